"""CPU tests of the library's host side: the C-ABI surface, batch-norm merge,
filter selection, filter removal, packing, model planning and error paths.
No kernel is launched here."""
import ctypes as C
import os
import re
import subprocess
import threading

import numpy as np
import pytest

import synth
from oracle import reference as orc
from paper_2010_16165_amd import binding as B, network

RNG = np.random.default_rng(3)
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def rand_bn(k):
    f = lambda a: np.asarray(a, dtype=np.float32)
    return {"gamma": f(RNG.uniform(0.5, 1.5, k)), "beta": f(RNG.standard_normal(k) * 0.1),
            "mean": f(RNG.standard_normal(k) * 0.1), "var": f(RNG.uniform(0.5, 1.5, k)), "eps": 1e-5}


# ---- C ABI surface ------------------------------------------------------------

def declared_in(header_name):
    header = open(os.path.join(ROOT, "include", header_name)).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    return set(re.findall(r"\b(fupr_[a-z_0-9]+)\s*\(", header))


def test_library_exports_every_declared_symbol():
    declared = declared_in("fupr.h")
    assert len(declared) >= 20
    lib = C.CDLL(B.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name
    assert declared == set(B.SIGNATURES), declared ^ set(B.SIGNATURES)


def test_measuring_library_exports_every_declared_symbol():
    """The measuring kernels live in a library of their own, apart from the product's."""
    from paper_2010_16165_amd import measure as M
    declared = declared_in("fupr_measure.h")
    assert declared == set(M.SIGNATURES) == {"fupr_measure_mfma", "fupr_measure_copy"}
    lib = C.CDLL(M.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name
    product = C.CDLL(B.LIB_PATH)
    assert not any(hasattr(product, name) for name in declared)


def test_library_owns_no_device_memory_or_stream():
    """Every device buffer and stream is the caller's: the product sources call no
    allocating, copying or stream-creating runtime routine."""
    csrc = os.path.join(ROOT, "paper_2010_16165_amd", "csrc")
    banned = re.compile(r"\bhip(Malloc\w*|Free\w*|Memcpy\w*|Memset\w*|StreamCreate\w*|HostMalloc|ExtMalloc\w*)\s*\(")
    for name in sorted(os.listdir(csrc)):
        text = open(os.path.join(csrc, name)).read()
        text = re.sub(r"//.*", "", text)
        hits = banned.findall(text)
        assert not hits, (name, hits)


def build_host_model(plan, base):
    return network.build(plan, base_address=base)


def test_tuning_switches():
    B.fupr_tuning_set("patch_tile", 4)
    B.fupr_tuning_set("patch_tile", None)
    B.fupr_tuning_set("conv_tile", "conv16t_64x16")
    B.fupr_tuning_set("conv_tile", "")
    for name in ("pipe_tile", "pipe_order", "stream_tile", "stream_blocks", "pair_filters", "split",
                 "conv_patch", "conv1x1_stream", "conv1x1_pipe", "conv1x1_fuse", "res_item", "debug"):
        B.fupr_tuning_set(name, 1)
        B.fupr_tuning_set(name, None)
    for gone in ("block_fuse", "block_tile"):      # switches of a kernel that was never built
        with pytest.raises(B.FuprError):
            B.fupr_tuning_set(gone, 1)
    with pytest.raises(B.FuprError) as e:
        B.fupr_tuning_set("no_such_switch", 1)
    assert e.value.status == B.ERR_ARG
    with pytest.raises(B.FuprError) as e:
        B.fupr_tuning_set("split", "9" * 200)
    assert e.value.status == B.ERR_ARG
    assert B._lib.fupr_tuning_set(None, None) == B.ERR_NULL


def test_one_kernel_table_is_the_callers():
    """The one-kernel schedule's table is written on the host for a device address
    the caller names; without one the model runs a kernel per operator."""
    model = synth.make_cifar_resnet(5, "bf16", 2, 400)
    plan = network.optimise(model)
    # host-only: made-up 256-byte aligned "device" addresses, nothing is dereferenced here
    base = 1 << 20
    m, _ = build_host_model(plan, base)
    nbytes = B._lib.fupr_model_table_bytes(m._h)
    assert nbytes > 0 and nbytes % 256 == 0
    assert m.num_launches == m.num_ops            # no table yet: per operator
    img_a = np.zeros(nbytes, np.uint8)
    img_b = np.zeros(nbytes, np.uint8)
    st = B._lib.fupr_model_table_write(m._h, C.c_void_p(1 << 30), img_a.ctypes.data_as(C.c_void_p))
    assert st == B.FUPR_OK
    st = B._lib.fupr_model_table_write(m._h, C.c_void_p((1 << 30) + 4096), img_b.ctypes.data_as(C.c_void_p))
    assert st == B.FUPR_OK
    assert not np.array_equal(img_a, img_b)       # the image holds addresses inside itself
    assert B._lib.fupr_model_table_write(m._h, C.c_void_p((1 << 30) + 8), img_a.ctypes.data_as(C.c_void_p)) == B.ERR_ALIGN
    assert B._lib.fupr_model_table_write(m._h, None, img_a.ctypes.data_as(C.c_void_p)) == B.ERR_NULL
    assert B._lib.fupr_model_set_table(m._h, C.c_void_p(1 << 30)) == B.FUPR_OK
    assert m.num_launches == 1
    assert B._lib.fupr_model_set_table(m._h, None) == B.FUPR_OK
    assert m.num_launches == m.num_ops
    # a network with a max-pool has no such table
    big = synth.make_imagenet_basic_resnet(13, "bf16", (1, 1, 1, 1), 300, widths=(4, 8, 8, 12), size=32, classes=7)
    mb, _ = build_host_model(network.optimise(big), base)
    assert B._lib.fupr_model_table_bytes(mb._h) == 0
    assert B._lib.fupr_model_set_table(mb._h, C.c_void_p(1 << 30)) == B.ERR_ARG
    assert B._lib.fupr_model_table_bytes(None) == 0


def test_side_streams_argument_checks():
    model = synth.make_cifar_resnet(5, "bf16", 1, 400)
    m, _ = build_host_model(network.optimise(model), 1 << 20)
    arr = (C.c_void_p * 4)(None, None, None, None)
    assert B._lib.fupr_model_set_side_streams(m._h, 0, None) == B.FUPR_OK
    assert B._lib.fupr_model_set_side_streams(m._h, 1, None) == B.ERR_NULL
    assert B._lib.fupr_model_set_side_streams(m._h, 1, arr) == B.ERR_NULL      # NULL stream
    assert B._lib.fupr_model_set_side_streams(m._h, 4, arr) == B.ERR_ARG
    assert B._lib.fupr_model_set_side_streams(m._h, -1, arr) == B.ERR_ARG
    assert B._lib.fupr_model_set_side_streams(None, 0, None) == B.ERR_NULL


def test_status_strings():
    for code in range(0, -12, -1):
        assert B.status_str(code) not in ("", "unknown status")
    assert B.status_str(-99) == "unknown status"


# ---- fold (Eq. 3-5 and the merge) -------------------------------------------------

def test_fold_matches_closed_form():
    w = RNG.standard_normal((6, 5, 3, 3)).astype(np.float32)
    bn = rand_bn(6)
    sh = B.shape_of(w, 1, 1)
    wf, bf = B.fupr_fold(sh, w, None, bn["gamma"], bn["beta"], bn["mean"], bn["var"], bn["eps"],
                         B.FUSE_BN)
    wo, bo = orc.fold(w, bn)
    assert wf.dtype == np.float32 and bf.dtype == np.float32
    np.testing.assert_allclose(wf, wo, rtol=2 ** -23)
    np.testing.assert_allclose(bf, bo, rtol=2 ** -22, atol=1e-9)


def test_fold_then_conv_equals_conv_then_bn():
    x = RNG.standard_normal((2, 5, 7, 7))
    w = RNG.standard_normal((6, 5, 3, 3)).astype(np.float32)
    bn = rand_bn(6)
    cb = RNG.standard_normal(6).astype(np.float32)
    sh = B.shape_of(w, 1, 1)
    wf, bf = B.fupr_fold(sh, w, cb, bn["gamma"], bn["beta"], bn["mean"], bn["var"], bn["eps"],
                         B.FUSE_BN)
    ref = orc.batchnorm(orc.conv2d(x, w, 1, 1) + cb[None, :, None, None].astype(np.float64), bn)
    got = orc.conv2d(x, wf, 1, 1) + bf[None, :, None, None].astype(np.float64)
    assert np.abs(got - ref).max() / np.abs(ref).max() <= 1e-5


def test_fold_identity_special_case_is_exact():
    k = 4
    var = RNG.uniform(0.5, 1.5, k).astype(np.float32)
    mean = RNG.standard_normal(k).astype(np.float32)
    # gamma = sqrt(var + eps) in double, eps = 0 so that omega is exactly 1 for perfect squares
    var = (np.arange(1, k + 1, dtype=np.float32)) ** 2
    gamma = np.arange(1, k + 1, dtype=np.float32)
    w = RNG.standard_normal((k, 3, 3, 3)).astype(np.float32)
    sh = B.shape_of(w, 1, 1)
    wf, bf = B.fupr_fold(sh, w, None, gamma, mean, mean, var, 0.0, B.FUSE_BN)
    assert np.array_equal(wf, w) and np.all(bf == 0)


def test_fold_without_bn_flag_copies():
    w = RNG.standard_normal((3, 2, 1, 1)).astype(np.float32)
    b = RNG.standard_normal(3).astype(np.float32)
    sh = B.shape_of(w, 1, 0)
    wf, bf = B.fupr_fold(sh, w, b, None, None, None, None, 1e-5, 0)
    assert np.array_equal(wf, w) and np.array_equal(bf, b)
    wf, bf = B.fupr_fold(sh, w, None, None, None, None, None, 1e-5, B.FUSE_RELU)
    assert np.all(bf == 0)


def expect(code, fn):
    with pytest.raises(B.FuprError) as e:
        fn()
    assert e.value.status == code, (e.value.status, code)


def test_fold_errors_leave_outputs_untouched():
    w = np.ones((2, 2, 1, 1), dtype=np.float32)
    bn = rand_bn(2)
    sh = B.shape_of(w, 1, 0)
    bad_var = np.array([1.0, -1.0], dtype=np.float32)
    expect(B.ERR_BN_VAR, lambda: B.fupr_fold(sh, w, None, bn["gamma"], bn["beta"], bn["mean"],
                                             bad_var, 1e-5, B.FUSE_BN))
    expect(B.ERR_BN_VAR, lambda: B.fupr_fold(sh, w, None, bn["gamma"], bn["beta"], bn["mean"],
                                             np.array([1.0, np.inf], dtype=np.float32), 1e-5,
                                             B.FUSE_BN))
    expect(B.ERR_NULL, lambda: B.fupr_fold(sh, w, None, None, bn["beta"], bn["mean"], bn["var"],
                                           1e-5, B.FUSE_BN))
    expect(B.ERR_ARG, lambda: B.fupr_fold(sh, w, None, bn["gamma"], bn["beta"], bn["mean"],
                                          bn["var"], 1e-5, 128))
    expect(B.ERR_SHAPE, lambda: B.fupr_fold(B.conv_shape(0, 2, 1, 1, 1, 0), w, None, bn["gamma"],
                                            bn["beta"], bn["mean"], bn["var"], 1e-5, B.FUSE_BN))
    # raw call: outputs keep their sentinel on error
    wout = np.full(4, 9.0, dtype=np.float32)
    bout = np.full(2, 9.0, dtype=np.float32)
    F = B._F
    st = B._lib.fupr_fold(C.byref(sh), w.ctypes.data_as(F), None, bn["gamma"].ctypes.data_as(F),
                          bn["beta"].ctypes.data_as(F), bn["mean"].ctypes.data_as(F),
                          bad_var.ctypes.data_as(F), C.c_float(1e-5), B.FUSE_BN,
                          wout.ctypes.data_as(F), bout.ctypes.data_as(F))
    assert st == B.ERR_BN_VAR and np.all(wout == 9.0) and np.all(bout == 9.0)


# ---- filter selection ------------------------------------------------------------------

@pytest.mark.parametrize("n,permille", [(16, 250), (16, 400), (32, 400), (64, 400), (64, 300),
                                        (128, 300), (256, 300), (512, 300), (64, 500), (4, 1000),
                                        (7, 0), (1, 999), (2048, 137)])
def test_prune_count_matches_oracle(n, permille):
    assert B.fupr_prune_count(n, permille) == orc.prune_count(n, permille)


def test_prune_count_errors():
    expect(B.ERR_ARG, lambda: B.fupr_prune_count(0, 100))
    expect(B.ERR_ARG, lambda: B.fupr_prune_count(8, 1001))
    expect(B.ERR_ARG, lambda: B.fupr_prune_count(8, -1))


@pytest.mark.parametrize("norm", [1, 2])
def test_select_filters_bit_exact_vs_oracle(norm):
    for k, c, r in [(16, 16, 3), (64, 3, 7), (39, 64, 3), (256, 64, 1), (5, 1, 1)]:
        w = RNG.standard_normal((k, c, r, r)).astype(np.float32)
        for n_prune in (0, 1, k // 3, k - 1):
            got = B.fupr_select_filters(B.shape_of(w, 1, 0), w, norm, n_prune)
            assert np.array_equal(got, orc.select_mask(w, n_prune, norm))
            assert int(got.sum()) == k - n_prune


def test_select_filters_tie_rule_and_norm_choice():
    w = np.ones((6, 2, 3, 3), dtype=np.float32)
    assert list(B.fupr_select_filters(B.shape_of(w, 1, 1), w, 1, 2)) == [0, 0, 1, 1, 1, 1]
    w = np.zeros((2, 4, 1, 1), dtype=np.float32)
    w[0, :, 0, 0] = 1
    w[1, 0, 0, 0] = 3
    sh = B.shape_of(w, 1, 0)
    assert list(B.fupr_select_filters(sh, w, 1, 1)) == [1, 0]
    assert list(B.fupr_select_filters(sh, w, 2, 1)) == [0, 1]
    expect(B.ERR_ARG, lambda: B.fupr_select_filters(sh, w, 3, 1))
    expect(B.ERR_ARG, lambda: B.fupr_select_filters(sh, w, 1, 2))
    expect(B.ERR_ARG, lambda: B.fupr_select_filters(sh, w, 1, -1))


@pytest.mark.parametrize("idx", [0, 1, 2, 3, 4])
def test_masks_of_baseline_configs_match_oracle(idx):
    model, _ = synth.make_config(idx)
    plan = network.optimise(model)
    masks = orc.select_masks(model)
    assert set(plan["masks"]) == set(masks) and masks
    for key, m in masks.items():
        assert np.array_equal(plan["masks"][key], m)
        assert np.array_equal(plan["keep_idx"][key], np.flatnonzero(m))
        assert plan["keep_idx"][key].dtype == np.int32


# ---- filter removal -----------------------------------------------------------------------

def test_prune_is_an_exact_gather():
    wp = RNG.standard_normal((9, 4, 3, 3)).astype(np.float32)
    bp = RNG.standard_normal(9).astype(np.float32)
    wc1 = RNG.standard_normal((7, 9, 3, 3)).astype(np.float32)
    wc2 = RNG.standard_normal((5, 9, 1, 1)).astype(np.float32)
    mask = np.array([1, 0, 1, 1, 0, 0, 1, 0, 1], dtype=np.uint8)
    keep, wpo, bpo, (w1o, w2o) = B.fupr_prune(B.shape_of(wp, 1, 1), wp, bp, mask,
                                              [B.shape_of(wc1, 1, 1), B.shape_of(wc2, 2, 0)],
                                              [wc1, wc2])
    idx = [0, 2, 3, 6, 8]
    assert list(keep) == idx
    # gather written out by hand
    for j, k in enumerate(idx):
        assert wpo[j].tobytes() == wp[k].tobytes() and bpo[j] == bp[k]
        for f in range(7):
            assert w1o[f, j].tobytes() == wc1[f, k].tobytes()
        for f in range(5):
            assert w2o[f, j].tobytes() == wc2[f, k].tobytes()
    assert wpo.shape == (5, 4, 3, 3) and w1o.shape == (7, 5, 3, 3) and w2o.shape == (5, 5, 1, 1)


def test_prune_without_bias_or_consumers():
    wp = RNG.standard_normal((4, 2, 1, 1)).astype(np.float32)
    keep, wpo, bpo, rest = B.fupr_prune(B.shape_of(wp, 1, 0), wp, None, [0, 1, 1, 0], [], [])
    assert list(keep) == [1, 2] and bpo is None and rest == [] and np.array_equal(wpo, wp[1:3])


def test_prune_and_fold_commute():
    """Per-filter scaling commutes with the gather: bit-exact either way round."""
    w1 = RNG.standard_normal((8, 3, 3, 3)).astype(np.float32)
    w2 = RNG.standard_normal((6, 8, 3, 3)).astype(np.float32)
    bn1, bn2 = rand_bn(8), rand_bn(6)
    s1, s2 = B.shape_of(w1, 1, 1), B.shape_of(w2, 1, 1)
    mask = B.fupr_select_filters(s1, w1, 1, 3)
    fold = lambda sh, w, bn: B.fupr_fold(sh, w, None, bn["gamma"], bn["beta"], bn["mean"],
                                         bn["var"], bn["eps"], B.FUSE_BN)
    # fold, then prune
    w1f, b1f = fold(s1, w1, bn1)
    w2f, b2f = fold(s2, w2, bn2)
    _, a1, ab1, (a2,) = B.fupr_prune(s1, w1f, b1f, mask, [s2], [w2f])
    # prune, then fold
    keep, p1, _, (p2,) = B.fupr_prune(s1, w1, None, mask, [s2], [w2])
    bn1k = {k: (v[keep] if k != "eps" else v) for k, v in bn1.items()}
    c1, cb1 = fold(B.shape_of(p1, 1, 1), p1, bn1k)
    c2, _ = fold(B.shape_of(p2, 1, 1), p2, bn2)
    assert np.array_equal(a1, c1) and np.array_equal(ab1, cb1) and np.array_equal(a2, c2)


def test_prune_errors():
    wp = np.ones((4, 2, 1, 1), dtype=np.float32)
    sh = B.shape_of(wp, 1, 0)
    wc = np.ones((3, 4, 1, 1), dtype=np.float32)
    expect(B.ERR_MASK_EMPTY, lambda: B.fupr_prune(sh, wp, None, [0, 0, 0, 0], [], []))
    expect(B.ERR_ARG, lambda: B.fupr_prune(sh, wp, None, [1, 2, 0, 0], [], []))
    bad = B.conv_shape(3, 5, 1, 1, 1, 0)     # consumer C != producer K
    expect(B.ERR_SHAPE, lambda: B.fupr_prune(sh, wp, None, [1, 1, 0, 0], [bad], [wc]))


def test_library_compaction_equals_oracle_extraction():
    """The thinner model the library builds is the oracle's `extract` of the
    merged weights, filter for filter."""
    model = synth.make_imagenet_bottleneck_resnet(14, "bf16", (2, 1, 1, 1), 500, widths=(4, 4, 8, 8),
                                                  size=32, classes=5)
    plan = network.optimise(model, concat_projection=False)
    thin = orc.extract(model, orc.select_masks(model))
    by_site = {L.site: L for L in plan["layers"]}
    for bi, blk in enumerate(thin["blocks"]):
        for ci, (conv, bn) in enumerate(zip(blk["convs"], blk["bns"])):
            L = by_site[f"b{bi}.conv{ci + 1}"]
            wo, bo = orc.fold(conv["W"], bn)
            assert L.W.shape == wo.shape
            np.testing.assert_allclose(L.W, wo, rtol=2 ** -23)
            np.testing.assert_allclose(L.bias, bo, rtol=2 ** -22, atol=1e-9)


# ---- packing ---------------------------------------------------------------------------------

def bf16_bits_rne(a):
    u = np.asarray(a, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = u + 0x7FFF + ((u >> 16) & 1)
    return (u >> 16).astype(np.uint16)


@pytest.mark.parametrize("k,c,r", [(10, 16, 3), (16, 10, 3), (64, 3, 7), (39, 64, 3), (1000, 20, 1),
                                   (1, 1, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_pack_16bit_layout(k, c, r, dtype):
    w = RNG.standard_normal((k, c, r, r)).astype(np.float32)
    b = RNG.standard_normal(k).astype(np.float32)
    sh = B.shape_of(w, 1, r // 2)
    blob = B.fupr_pack(sh, w, b, B.DTYPES[dtype])
    kp, cp = (k + 15) // 16 * 16, (c + 7) // 8 * 8
    nchunk = r * r * cp // 8
    nchunk_pad = (nchunk + 3) // 4 * 4
    woff = (kp * 4 + 255) // 256 * 256
    assert len(blob) == (woff + nchunk_pad * kp * 16 + 255) // 256 * 256 == B.fupr_packed_bytes(
        sh, B.DTYPES[dtype])
    bias = blob[:kp * 4].view(np.float32)
    assert np.array_equal(bias[:k], b) and np.all(bias[k:] == 0)
    wt = blob[woff:woff + nchunk_pad * kp * 16].view(np.uint16).reshape(nchunk_pad, kp, 8)
    expect_bits = np.zeros((nchunk_pad, kp, 8), dtype=np.uint16)
    bits = bf16_bits_rne(w) if dtype == "bf16" else w.astype(np.float16).view(np.uint16)
    for rr in range(r):
        for ss in range(r):
            for cc in range(c):
                expect_bits[(rr * r + ss) * (cp // 8) + cc // 8, :k, cc % 8] = bits[:, cc, rr, ss]
    assert np.array_equal(wt, expect_bits)


def test_pack_16bit_rounding_edge_cases():
    vals = np.array([1.0, 1.00390625, 1.01171875, 65519.9, 65520.0, 1e-8, 5.96e-8, 6.1e-5, -0.0,
                     3.0e-5, np.inf, 70000.0], dtype=np.float32)
    w = np.zeros((1, 16, 1, 1), dtype=np.float32)
    w[0, :len(vals), 0, 0] = vals
    sh = B.shape_of(w, 1, 0)
    for dtype in ("bf16", "f16"):
        blob = B.fupr_pack(sh, w, None, B.DTYPES[dtype])
        wt = blob[256:256 + 4 * 16 * 16].view(np.uint16).reshape(4, 16, 8)
        got = np.concatenate([wt[0, 0], wt[1, 0]])
        with np.errstate(over="ignore"):
            want = bf16_bits_rne(w[0, :, 0, 0]) if dtype == "bf16" else \
                w[0, :, 0, 0].astype(np.float16).view(np.uint16)
        assert np.array_equal(got, want), dtype


def test_pack_f32_layout():
    k, c, r = 10, 6, 3
    w = RNG.standard_normal((k, c, r, r)).astype(np.float32)
    sh = B.shape_of(w, 1, 1)
    blob = B.fupr_pack(sh, w, None, B.F32)
    kp, cp = 12, 8
    assert len(blob) == 256 + (r * r * cp * kp * 4 + 255) // 256 * 256
    assert np.all(blob[:kp * 4].view(np.float32) == 0)
    wt = blob[256:256 + r * r * cp * kp * 4].view(np.float32).reshape(r * r, cp, kp)
    want = np.zeros((r * r, cp, kp), dtype=np.float32)
    want[:, :c, :k] = w.transpose(2, 3, 1, 0).reshape(r * r, c, k)
    assert np.array_equal(wt, want)


def test_pack_errors():
    assert B.fupr_packed_bytes(B.conv_shape(0, 1, 1, 1, 1, 0), B.BF16) == 0
    assert B.fupr_packed_bytes(B.conv_shape(1, 1, 1, 1, 1, 0), 7) == 0
    w = np.zeros((1, 1, 1, 1), dtype=np.float32)
    st = B._lib.fupr_pack(C.byref(B.conv_shape(1, 1, 1, 1, 1, 0)), w.ctypes.data_as(B._F), None, 7,
                          C.c_void_p(w.ctypes.data))
    assert st == B.ERR_DTYPE
    st = B._lib.fupr_pack(C.byref(B.conv_shape(1, 1, 1, 1, 1, 0)), None, None, B.BF16,
                          C.c_void_p(w.ctypes.data))
    assert st == B.ERR_NULL


# ---- model planning (host only; device pointers are never dereferenced) -----------------------

def fake_ops(specs):
    """specs: (kind, in, res, K, C, R, stride, pad, epilogue, rss)"""
    ops = []
    for kind, tin, res, k, c, r, st, pd, epi, rss in specs:
        ops.append(B.OpDesc(kind, tin, res, B.conv_shape(k, c, r, r, st, pd), 0x1000, epi, rss, 0))
    return ops


def test_model_plan_shares_buffers_and_reports_shapes():
    ops = fake_ops([
        (B.OP_CONV, 0, -1, 16, 3, 3, 1, 1, B.FUSE_RELU, 1),                  # t1 16x32x32
        (B.OP_CONV, 1, -1, 10, 16, 3, 1, 1, B.FUSE_RELU, 1),                 # t2
        (B.OP_CONV, 2, 1, 16, 10, 3, 1, 1, B.FUSE_RELU | B.FUSE_ADD, 1),     # t3 (+t1)
        (B.OP_CONV, 3, -1, 20, 16, 3, 2, 1, B.FUSE_RELU, 1),                 # t4 20x16x16
        (B.OP_CONV, 4, 3, 32, 20, 3, 1, 1, B.FUSE_RELU | B.FUSE_ADD, 2),     # t5 32x16x16 (+t3 ::2)
        (B.OP_AVGPOOL, 5, -1, 1, 1, 1, 1, 0, 0, 1),
        (B.OP_CONV, 6, -1, 10, 32, 1, 1, 0, 0, 1),
    ])
    m = B.Model(B.BF16, (3, 32, 32), ops, None)
    assert m.num_ops == 7
    t = m.output_shape(5)
    assert (t.N, t.H, t.W, t.C, t.c_stride) == (5, 1, 1, 10, 16)
    # three live 16-channel 32x32 tensors at most -> three buffers of 32 KB per image
    assert m.workspace_bytes(1) == 3 * 32 * 32 * 16 * 2
    assert m.workspace_bytes(4) == 4 * m.workspace_bytes(1)
    s = m.op_stats(2, 2)
    assert s["flops"] == 2.0 * 10 * 9 * 16 * 2 * 1024
    assert s["bytes"] == 2 * (2 * 1024 * 10 + 2 * 1024 * 16 + 2 * 1024 * 16 + 16 * 10 * 9) + 4 * 16
    assert s["kernel"].startswith("conv")


def test_input_of_a_stem_with_its_pool_outlives_the_launch():
    """A 7 x 7 convolution and its max-pool run as one kernel wherever they stand: the pool's output is
    written while other workgroups still read the convolution's input, so the two share no buffer."""
    ops = fake_ops([
        (B.OP_CONV, 0, -1, 3, 3, 1, 1, 0, B.FUSE_RELU, 1),                   # t1 3x64x64
        (B.OP_CONV, 1, -1, 64, 3, 7, 2, 3, B.FUSE_RELU, 1),                  # t2 64x32x32
        (B.OP_MAXPOOL, 2, -1, 64, 64, 3, 2, 1, 0, 1),                        # t3 64x16x16
        (B.OP_CONV, 3, -1, 10, 64, 1, 1, 0, 0, 1),
    ])
    m = B.Model(B.BF16, (3, 64, 64), ops, None)
    assert [m.launch_stats(1, i)["kernel"] for i in range(m.num_launches_at(1))][1] == "stem7x7_maxpool"
    assert m.workspace_bytes(1) == 2 * (64 * 64 * 8 + 32 * 32 * 64 + 16 * 16 * 64)
    # ... and a stem that reads the network's input needs no more than its two tensors
    m = B.Model(B.BF16, (3, 64, 64), [B.OpDesc(o.kind, o.in_ - 1, -1, o.conv, 0x1000, o.epilogue, 1, 0) for o in ops[1:]],
                None)
    assert m.workspace_bytes(1) == 2 * (32 * 32 * 64 + 16 * 16 * 64)


def test_kernel_selection_per_layer_class():
    """Which kernel an operator launches is decided on the host from its shape
    alone: every layer class of the ImageNet workloads must get its own kernel."""
    ops = fake_ops([
        (B.OP_CONV, 0, -1, 64, 3, 7, 2, 3, B.FUSE_RELU, 1),                   # t1 64 x 112 x 112
        (B.OP_MAXPOOL, 1, -1, 1, 1, 3, 2, 1, 0, 1),                           # t2 64 x 56 x 56
        (B.OP_CONV, 2, -1, 45, 64, 3, 1, 1, B.FUSE_RELU, 1),                  # t3
        (B.OP_CONV, 3, 2, 64, 45, 3, 1, 1, B.FUSE_RELU | B.FUSE_ADD, 1),      # t4
        (B.OP_CONV, 4, -1, 256, 64, 1, 1, 0, 0, 1),                           # t5 256 x 56 x 56
        (B.OP_CONV, 5, -1, 32, 256, 1, 1, 0, B.FUSE_RELU, 1),                 # t6
        (B.OP_CONV, 6, -1, 90, 32, 3, 2, 1, B.FUSE_RELU, 1),                  # t7 90 x 28 x 28
        (B.OP_CONV, 7, -1, 1024, 90, 1, 2, 0, 0, 1),                          # t8 1024 x 14 x 14
        (B.OP_CONV, 8, -1, 128, 1024, 1, 1, 0, B.FUSE_RELU, 1),               # t9
    ])
    m = B.Model(B.BF16, (3, 224, 224), ops, None)
    names = [m.op_stats(64, i)["kernel"] for i in range(m.num_ops)]
    assert names[2].startswith("conv3x3p_") and names[3].startswith("conv3x3p_")
    assert names[4].startswith("conv1x1s_") and names[5].startswith("conv1x1s_")
    assert names[6].startswith("conv16t_")        # stride 2 at 56 x 56: the general kernel
    assert names[8].startswith("conv1x1p_")       # 1024 channels: filters do not fit in LDS
    # the stem convolution and the max-pool behind it are one launch, and so are
    # the 64 -> 256 and 256 -> 32 1 x 1 convolutions (the second from the first's registers)
    assert m.num_launches == m.num_ops - 2
    pair = m.launch_stats(64, 3)
    a, b = m.op_stats(64, 4), m.op_stats(64, 5)
    assert pair["kernel"] == "conv1x1s_256f+conv1x1" and pair["flops"] == a["flops"] + b["flops"]
    assert pair["bytes"] == a["bytes"] + b["bytes"] - 2 * 64 * 56 * 56 * 256
    first = m.launch_stats(64, 0)
    assert first["kernel"] == "stem7x7_maxpool"
    conv, pool = m.op_stats(64, 0), m.op_stats(64, 1)
    mid = 2 * 64 * 112 * 112 * 64
    assert first["flops"] == conv["flops"] and first["bytes"] == conv["bytes"] + pool["bytes"] - 2 * mid
    m.set_schedule(B.SCHEDULE_PER_LAYER)
    assert m.num_launches == m.num_ops and m.launch_stats(64, 0)["kernel"].startswith("conv16t_")


def conv_name(dtype, n, c, h, w, k, r, s, stride, pad):
    """The kernel one convolution operator launches at a batch of n images."""
    op = B.OpDesc(B.OP_CONV, 0, -1, B.conv_shape(k, c, r, s, stride, pad), 0x1000, 0, 1, 0)
    return B.Model(dtype, (c, h, w), [op], None).op_stats(n, 0)["kernel"]


# padding beyond half a window on its shorter side, with the sides that a window needs for it
WIDE_PADDING = [(1, 128, 14, 14, 64, 3, 3, 1, 2), (1, 256, 56, 56, 64, 3, 3, 1, 2), (2, 64, 14, 14, 64, 3, 3, 1, 3),
                (1, 64, 30, 42, 16, 3, 3, 1, 2), (1, 256, 14, 14, 64, 1, 1, 1, 1), (1, 256, 14, 14, 64, 1, 1, 2, 2),
                (1, 128, 28, 28, 64, 5, 5, 1, 4), (3, 64, 8, 12, 32, 1, 3, 1, 1), (3, 64, 8, 12, 32, 5, 1, 1, 2)]


@pytest.mark.parametrize("dtype", [B.BF16, B.F16, B.F32])
def test_paddings_over_half_a_window_stay_off_the_window_kernel(dtype):
    """That kernel fills LDS with one run of input pixels per tile, which holds every tap only up to
    half a window of padding: other layers go to the kernels that look every tap up by itself."""
    for case in WIDE_PADDING:
        assert "_w" not in conv_name(dtype, *case), case
    for case in [(1, 64, 14, 14, 64, 3, 3, 1, 1), (1, 64, 14, 14, 64, 2, 2, 1, 1), (1, 64, 14, 14, 64, 5, 5, 1, 2),
                 (1, 64, 14, 14, 64, 3, 5, 1, 1), (1, 64, 14, 14, 64, 1, 3, 1, 0)]:
        assert "_w" in conv_name(dtype, *case), case


def test_weights_of_2_gib_and_more_stay_off_the_window_kernel():
    """That kernel reads weights through 32-bit offsets; the fp32 kernel that takes such layers does not."""
    for dtype, c, k, takes in [(B.F32, 2048, 1 << 17, True), (B.F32, 2048, (1 << 18) - 16, True),
                               (B.F32, 2048, 1 << 18, False), (B.F32, 2048, 1 << 19, False),
                               (B.F32, 2052, (1 << 19) - 4, False), (B.BF16, 1024, (1 << 20) - 16, True),
                               (B.BF16, 1024, 1 << 20, False), (B.BF16, 1024, (1 << 21) - 16, False)]:
        name = conv_name(dtype, 1, c, 1, 1, k, 1, 1, 1, 0)
        assert ("_w" in name) == takes, (dtype, c, k, name)
        assert takes or dtype != B.F32 or name == "conv32_direct"


def test_window_runs_hold_every_tap_and_fit_their_plan(tmp_path):
    """The functions the planner and the kernel share, walked tile by tile on the host."""
    exe = str(tmp_path / "window_runs")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2010_16165_amd", "csrc"),
                    os.path.join(ROOT, "tests", "window_runs.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert int(out.stdout) > 100000


def one_kernel_of(in_shape, specs):
    """The kernel of a whole network's one launch, "" where it has none (the table is never read here)."""
    m = B.Model(B.BF16, in_shape, fake_ops(specs), None)
    if B._lib.fupr_model_set_table(m._h, B.C.c_void_p(1 << 20)) != B.FUPR_OK or m.num_launches != 1:
        return ""
    return m.launch_stats(2, 0)["kernel"]


def network_of(c, layers, classes=10):
    """3 x 3 convolutions (filters, stride, tensor that is added or -1, its stride), their mean and a layer behind it."""
    specs, width = [], c
    for i, (k, stride, add, add_stride) in enumerate(layers):
        specs.append((B.OP_CONV, i, add, k, width, 3, stride, 1, B.FUSE_RELU | (B.FUSE_ADD if add >= 0 else 0), add_stride))
        width = k
    specs.append((B.OP_AVGPOOL, len(layers), -1, 1, 1, 1, 1, 0, 0, 1))
    return specs + [(B.OP_CONV, len(layers) + 1, -1, classes, width, 1, 1, 0, 0, 1)]


ROWS, TAPS = "resident_network", "resident_network_taps"


@pytest.mark.parametrize("in_shape,layers,kernel", [
    ((3, 32, 32), [(16, 1, -1, 1), (16, 1, 1, 1)], ROWS),
    ((16, 6, 16), [(24, 1, -1, 1), (24, 1, 1, 1)], ROWS),      # not square
    ((8, 4, 48), [(16, 1, -1, 1), (16, 1, 1, 1)], ROWS),       # three tiles a row
    ((8, 2, 64), [(16, 1, -1, 1)], ROWS),                      # rows in pairs
    ((16, 8, 8), [(32, 1, -1, 1), (64, 1, -1, 1)], ROWS),      # tiles of two half rows
    ((16, 12, 8), [(32, 1, -1, 1), (24, 1, -1, 1)], ROWS),
    ((8, 12, 32), [(16, 1, -1, 1), (32, 2, -1, 1), (32, 1, 1, 2)], ROWS),
    ((16, 8, 16), [(64, 1, -1, 1)], ROWS),                     # eight work items of four filter tiles
    ((16, 16, 48), [(32, 1, -1, 1)], TAPS),                    # more work items than waves
    ((3, 24, 24), [(16, 1, -1, 1), (16, 1, 1, 1)], TAPS),      # rows of no whole tiles
    ((16, 7, 8), [(16, 1, -1, 1)], TAPS),                      # half rows of an odd number of rows
    ((16, 3, 16), [(16, 1, -1, 1)], TAPS),                     # an odd number of rows
    ((16, 16, 16), [(80, 1, -1, 1)], TAPS),                    # more than 64 filters
    ((40, 16, 32), [(16, 2, -1, 1)], TAPS),                    # a stride of 2 over more than 32 channels
])
def test_networks_of_row_layers(in_shape, layers, kernel):
    """Which networks the kernel of row layers takes, by their sizes, and that a switch leaves it out."""
    specs = network_of(in_shape[0], layers)
    assert one_kernel_of(in_shape, specs) == kernel
    B.fupr_tuning_set("resident_rows", 0)
    try:
        assert one_kernel_of(in_shape, specs) == TAPS
    finally:
        B.fupr_tuning_set("resident_rows", None)


def test_every_tile_of_two_convolutions_in_one_launch_is_taken_once(tmp_path):
    """The function by which a workgroup finds its tile, walked over grids that are larger than one of the two needs."""
    exe = str(tmp_path / "window_tiles")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2010_16165_amd", "csrc"),
                    os.path.join(ROOT, "tests", "window_tiles.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert int(out.stdout) > 20000


def test_launch_list_of_a_batch_names_what_runs():
    """A pair of 1 x 1 convolutions runs as two launches at batches whose tensors are small: the list of
    that batch counts both, under the kernels and bytes of the two operators."""
    ops = fake_ops([
        (B.OP_CONV, 0, -1, 64, 8, 1, 1, 0, B.FUSE_RELU, 1),
        (B.OP_CONV, 1, -1, 256, 64, 1, 1, 0, B.FUSE_RELU, 1),
        (B.OP_CONV, 2, -1, 32, 256, 1, 1, 0, B.FUSE_RELU, 1),
        (B.OP_CONV, 3, -1, 10, 32, 3, 1, 1, B.FUSE_RELU, 1),
    ])
    m = B.Model(B.F16, (8, 56, 56), ops, None)
    assert m.num_launches == m.num_launches_at(64) == 3 and m.num_launches_at(1) == 4
    for batch in (1, 3, 9, 64):
        n = m.num_launches_at(batch)
        launches = [m.launch_stats(batch, i) for i in range(n)]
        single = [m.op_stats(batch, i) for i in range(m.num_ops)]
        expect(B.ERR_ARG, lambda: m.launch_stats(batch, n))
        assert [i for s in launches for i in range(s["first_op"], s["first_op"] + s["n_ops"])] == list(range(4))
        assert sum(s["flops"] for s in launches) == sum(s["flops"] for s in single)
        paired = [s for s in launches if s["n_ops"] == 2]
        saved = 2 * batch * 56 * 56 * 256 * len(paired)    # the tensor in between is not read back
        assert sum(s["bytes"] for s in launches) == sum(s["bytes"] for s in single) - saved
        assert all(s["kernel"] == "conv1x1s_256f+conv1x1" for s in paired)
        assert all(s["kernel"] == single[s["first_op"]]["kernel"] for s in launches if s["n_ops"] == 1)
        # such a pair is split exactly where the window kernel takes its first convolution
        assert ("_w" in single[1]["kernel"]) == (not paired)
    m.set_schedule(B.SCHEDULE_PER_LAYER)
    assert m.num_launches == m.num_launches_at(64) == 4
    assert B._lib.fupr_model_num_launches_at(None, 4) == 0 and m.num_launches_at(0) == 0


@pytest.mark.parametrize("offset", [0, 4, 8, 12])
def test_shortcut_offset_decides_kernel_and_pairs(offset):
    """A 16-bit shortcut whose first channel is no multiple of 8 cannot be read 16 bytes at a time: such an
    operator runs on the general kernel, under that name, and never as the first half of a pair."""
    ops = fake_ops([
        (B.OP_CONV, 0, -1, 32, 8, 1, 1, 0, B.FUSE_RELU, 1),
        (B.OP_CONV, 1, 1, 64, 32, 3, 1, 1, B.FUSE_RELU | B.FUSE_ADD, 1),
        (B.OP_CONV, 2, 1, 256, 64, 1, 1, 0, B.FUSE_RELU | B.FUSE_ADD, 1),
        (B.OP_CONV, 3, -1, 32, 256, 1, 1, 0, B.FUSE_RELU, 1),
    ])
    for op in ops[1:3]:
        op.res_c_offset = offset
    m = B.Model(B.BF16, (8, 56, 56), ops, None)
    for batch in (1, 64):
        for i in (1, 2):
            name = m.op_stats(batch, i)["kernel"]
            general = name.startswith("conv16t_") and "_w" not in name
            # (the pipelined 1 x 1 kernel is not chosen at 64 images, and takes the offset where it is)
            assert general == (offset % 8 != 0), (batch, i, name)
    assert m.num_launches == m.num_launches_at(64) == (4 if offset % 8 else 3)


def test_model_create_errors():
    ok = (B.OP_CONV, 0, -1, 16, 3, 3, 1, 1, B.FUSE_RELU, 1)
    cases = [
        ([(B.OP_CONV, 0, -1, 16, 4, 3, 1, 1, 0, 1)], B.ERR_SHAPE),             # C mismatch
        ([ok, (B.OP_CONV, 2, -1, 16, 16, 3, 1, 1, 0, 1)], B.ERR_ARG),          # reads a later tensor
        ([ok, (B.OP_CONV, 1, 0, 16, 16, 3, 1, 1, 0, 1)], B.ERR_ARG),           # res without ADD
        ([ok, (B.OP_CONV, 1, -1, 16, 16, 3, 1, 1, B.FUSE_ADD, 1)], B.ERR_ARG),  # ADD without res
        ([ok, (B.OP_CONV, 1, 0, 16, 16, 3, 2, 1, B.FUSE_ADD, 3)], B.ERR_SHAPE),  # residual too small
        ([ok, (7, 1, -1, 1, 1, 1, 1, 0, 0, 1)], B.ERR_ARG),                    # unknown kind
        ([ok, (B.OP_MAXPOOL, 1, -1, 1, 1, 3, 2, 3, 0, 1)], B.ERR_ARG),         # pad >= window
        ([(B.OP_CONV, 0, -1, 16, 3, 40, 1, 1, 0, 1)], B.ERR_SHAPE),            # window larger than image
    ]
    for specs, code in cases:
        expect(code, lambda: B.Model(B.BF16, (3, 32, 32), fake_ops(specs), None))
    expect(B.ERR_DTYPE, lambda: B.Model(5, (3, 32, 32), fake_ops([ok]), None))
    bad = fake_ops([ok])
    bad[0].packed = None
    expect(B.ERR_NULL, lambda: B.Model(B.BF16, (3, 32, 32), bad, None))


def test_baseline_config_graphs_have_expected_launch_counts():
    want = {0: 2, 1: 56, 2: 21, 3: 54, 4: 54}
    for idx, n in want.items():
        model, _ = synth.make_config(idx)
        plan = network.optimise(model, concat_projection=False)
        assert len(plan["layers"]) == n
        # a bottleneck block's projection shortcut is part of its last convolution by default
        plan = network.optimise(model)
        assert len(plan["layers"]) == n - (4 if idx >= 3 else 0)
        assert sum(L.cat_stride > 0 for L in plan["layers"]) == (4 if idx >= 3 else 0)


def test_largest_workload_pairs_its_first_stage_output_with_the_next_convolution():
    """The launch list of the largest workload: stem + pool, three pairs of 1 x 1 convolutions in
    the first stage (the third with the 90-filter first convolution of the next stage), 48
    launches for 52 operators; with pairs limited to 64 second filters it has one more."""
    model, batch = synth.make_config(4)
    plan = network.optimise(model)
    m, _ = build_host_model(plan, 1 << 20)
    assert (m.num_ops, m.num_launches) == (52, 48)
    kernels = [m.launch_stats(batch, i)["kernel"] for i in range(m.num_launches)]
    assert kernels.count("conv1x1s_256f+conv1x1") == 3 and kernels[0] == "stem7x7_maxpool"
    B.fupr_tuning_set("pair_filters", 64)
    try:
        m2, _ = build_host_model(plan, 1 << 20)
        assert m2.num_launches == 49
    finally:
        B.fupr_tuning_set("pair_filters", None)


def test_blocks_run_as_one_launch_only_when_asked_for():
    """fupr_model_fuse_blocks changes the launches of a batch, never the list without a batch or the
    workspace; what a launch covers and does adds up to the operators."""
    model, _ = synth.make_config(3)
    m, _ = build_host_model(network.optimise(model), 1 << 20)
    m2, _ = build_host_model(network.optimise(model), 1 << 20)
    assert B._lib.fupr_model_fuse_blocks(None, 1) == B.ERR_NULL
    assert B._lib.fupr_model_fuse_blocks(m._h, 2) == B.ERR_ARG
    m.fuse_blocks(True)
    assert m.num_launches == m2.num_launches
    covered = set()
    for batch in (1, 3, 9, 24, 64, 256):
        assert m.workspace_bytes(batch) == m2.workspace_bytes(batch)
        launches = [m.launch_stats(batch, i) for i in range(m.num_launches_at(batch))]
        single = [m.op_stats(batch, i) for i in range(m.num_ops)]
        assert [i for s in launches for i in range(s["first_op"], s["first_op"] + s["n_ops"])] == list(range(m.num_ops))
        assert sum(s["flops"] for s in launches) == sum(s["flops"] for s in single)
        blocks = [s for s in launches if s["kernel"].startswith("bottleneck_")]
        covered |= {s["first_op"] for s in blocks}
        for s in blocks:
            a, b = s["first_op"], s["first_op"] + 1
            assert single[a]["R"] == 3 and single[b]["R"] == 1
            mid, y = ([2 * single[i]["M"] * single[i]["K"] for i in (a, b)])
            assert s["bytes"] == sum(single[i]["bytes"] for i in range(a, a + s["n_ops"])) - 2 * mid - y * (s["n_ops"] - 2)
        assert blocks and m2.num_launches_at(batch) == m.num_launches_at(batch) + sum(s["n_ops"] - 1 for s in blocks) \
            - sum(s["n_ops"] == 2 and s["kernel"].startswith("conv1x1s") for s in
                  (m2.launch_stats(batch, i) for i in range(m2.num_launches_at(batch)))) \
            + sum(s["n_ops"] == 2 and s["kernel"].startswith("conv1x1s") for s in launches)
    assert len(covered) >= 12         # of 16 blocks, at one batch or another
    m.set_schedule(B.SCHEDULE_PER_LAYER)
    assert m.num_launches_at(9) == m.num_ops
    m.set_schedule(B.SCHEDULE_AUTO)
    m.fuse_blocks(False)
    assert m.num_launches_at(9) == m2.num_launches_at(9)


@pytest.mark.parametrize("config,kinds", [(0, 1), (2, 4)])
def test_basic_blocks_run_as_one_launch(config, kinds):
    """Both 3 x 3 convolutions of a basic block, the block of a two-operator model included: what the launch
    does not write and read is the tensor between them."""
    model, _ = synth.make_config(config)
    m, _ = build_host_model(network.optimise(model), 1 << 20)
    m.fuse_blocks(True)
    covered = set()
    for batch in (1, 8, 64):
        launches = [m.launch_stats(batch, i) for i in range(m.num_launches_at(batch))]
        single = [m.op_stats(batch, i) for i in range(m.num_ops)]
        assert [i for s in launches for i in range(s["first_op"], s["first_op"] + s["n_ops"])] == list(range(m.num_ops))
        for s in launches:
            if not s["kernel"].startswith("basic_block_"):
                continue
            a, b = (single[i] for i in (s["first_op"], s["first_op"] + 1))
            assert s["n_ops"] == 2 and a["R"] == b["R"] == 3 and b["stride"] == 1
            size = 4 if config == 0 else 2
            assert s["flops"] == a["flops"] + b["flops"]
            assert s["bytes"] == a["bytes"] + b["bytes"] - 2 * size * a["M"] * a["K"]
            covered.add(s["first_op"])
    assert len(covered) >= kinds


def test_blocks_only_where_networks_gain_from_them():
    """Short single-precision blocks, basic blocks of batches that run as two sub-batches and 1 x 1
    convolutions that are no pair at small extents: slower in one launch inside a network, so apart."""
    def blocks(make, *args, batch, **kwargs):
        m, _ = build_host_model(network.optimise(make(3, *args, **kwargs)), 1 << 20)
        m.fuse_blocks(True)
        launches = [m.launch_stats(batch, i) for i in range(m.num_launches_at(batch))]
        return [s for s in launches if s["kernel"].startswith(("basic_block_", "bottleneck_"))]

    cifar = lambda n: blocks(synth.make_cifar_resnet, "f32", 3, 200, batch=n)
    assert [len(cifar(n)) for n in (1, 2, 4)] == [0, 0, 0]
    assert len(cifar(8)) == 3 and len(cifar(16)) >= 3 and len(cifar(32)) == 6
    # nothing before or behind the block: one launch less is what the caller waits for
    assert len(blocks(synth.make_block_model, "f32", 16, 32, 250, batch=1)) == 1
    basic = lambda n: blocks(synth.make_imagenet_basic_resnet, "bf16", (2, 2, 2, 2), 500, batch=n, size=96)
    assert basic(1) and basic(128) and not basic(192) and not basic(256)
    # the deepest stages: little but weights
    deep = [s for s in blocks(synth.make_imagenet_bottleneck_resnet, "f16", (3, 4, 6, 3), 300, batch=192, size=96)
            if s["M"] == 192 * 6 * 6 and s["n_ops"] == 3]
    assert not deep


@pytest.mark.parametrize("config", [2, 3, 4])
def test_kept_launch_list_is_the_one_made_anew(config):
    """The list of a batch, pairs of operators in one launch among it, is kept from the first look on; with a switch set
    that decides nothing here it is made anew, and one that splits the pairs is neither kept nor overlooked."""
    model, _ = synth.make_config(config)
    m, _ = build_host_model(network.optimise(model), 1 << 20)
    m.fuse_blocks(True)
    look = lambda n: [(s["first_op"], s["n_ops"], s["kernel"]) for s in
                      (m.launch_stats(n, i) for i in range(m.num_launches_at(n)))]
    batches = (1, 2, 9, 12, 20, 64, 200)
    kept = [look(n) for n in batches]
    pairs = {"conv_w+conv1x1p_w", "mean_fc"}
    if config == 2:
        assert {k for l in kept for _, _, k in l} >= pairs
    try:
        B.fupr_tuning_set("res_item", "1/1/1:1x1")
        assert [look(n) for n in batches] == kept
        for switch in ("conv_two", "mean_fc"):
            B.fupr_tuning_set(switch, 0)
        assert not pairs & {k for n in batches for _, _, k in look(n)}
    finally:
        for switch in ("res_item", "conv_two", "mean_fc"):
            B.fupr_tuning_set(switch, None)
    assert [look(n) for n in batches] == kept


def launch_list(m, batch):
    return [(s["first_op"], s["n_ops"], s["kernel"]) for s in (m.launch_stats(batch, i) for i in range(m.num_launches))]


@pytest.mark.parametrize("switch,value", [("conv1x1_fuse", 0), ("conv1x1_stream", 0), ("pair_filters", 16), ("split", 2)]
                         + [("stream_tile", t) for t in range(6)])
def test_switches_at_creation_leave_nothing_behind(switch, value):
    """A model created while a switch is set has, once the switch is cleared, the launches and the
    workspace of any other: pairs are planned by the layers alone.  While one is set, only pairs whose
    tensors the workspace keeps apart are launched together."""
    ops = lambda: fake_ops([
        (B.OP_CONV, 0, -1, 64, 8, 1, 1, 0, B.FUSE_RELU, 1),
        (B.OP_CONV, 1, -1, 256, 64, 1, 1, 0, B.FUSE_RELU, 1),                  # a pair
        (B.OP_CONV, 2, -1, 32, 256, 1, 1, 0, B.FUSE_RELU, 1),
        (B.OP_CONV, 3, -1, 100, 32, 1, 1, 0, B.FUSE_RELU, 1),                  # a pair only if its tile is forced
        (B.OP_CONV, 4, -1, 40, 100, 1, 1, 0, B.FUSE_RELU, 1),
        (B.OP_CONV, 5, -1, 10, 40, 3, 1, 1, B.FUSE_RELU, 1),
    ])
    plain = B.Model(B.BF16, (8, 56, 56), ops(), None)
    want, want_ws = launch_list(plain, 64), plain.workspace_bytes(64)
    assert plain.num_launches == plain.num_ops - 1
    B.fupr_tuning_set(switch, value)
    try:
        other = B.Model(B.BF16, (8, 56, 56), ops(), None)
        both = [(m.num_launches, m.workspace_bytes(64)) for m in (plain, other)]
        other.set_schedule(B.SCHEDULE_PER_LAYER)
        assert other.num_launches == other.num_ops
        other.set_schedule(B.SCHEDULE_AUTO)
    finally:
        B.fupr_tuning_set(switch, None)
    assert both[0] == both[1] and both[0][0] >= plain.num_launches
    for m in (plain, other):
        assert launch_list(m, 64) == want and m.workspace_bytes(64) == want_ws
        m.set_schedule(B.SCHEDULE_PER_LAYER)
        assert m.num_launches == m.num_ops


@pytest.mark.parametrize("switch,value", [("conv1x1_fuse", 0), ("conv1x1_stream", 0), ("pair_filters", 16)]
                         + [("stream_tile", t) for t in range(6)])
def test_switches_decide_pairs_beside_blocks(switch, value):
    """With blocks in one launch a batch lists a pair of 1 x 1 convolutions only where it does without
    them: one that the switches of the moment refuse would end the pass when it is reached."""
    plan = network.optimise(synth.make_config(3)[0])
    models = [build_host_model(plan, 1 << 20)[0] for _ in range(2)]
    models[0].fuse_blocks(True)
    B.fupr_tuning_set(switch, value)
    try:
        for batch in (9, 64, 256):
            with_blocks, without = ([m.launch_stats(batch, i) for i in range(m.num_launches_at(batch))] for m in models)
            assert any(s["kernel"].startswith("bottleneck_") for s in with_blocks)
            pairs = [{(s["first_op"], s["kernel"]) for s in v if s["n_ops"] == 2 and s["kernel"].startswith("conv1x1s")}
                     for v in (with_blocks, without)]
            assert pairs[0] <= pairs[1]
    finally:
        B.fupr_tuning_set(switch, None)


def test_switches_set_meanwhile_are_in_no_list_that_is_kept():
    """A list that is worked out with no switch set is kept: one that another thread sets at that moment has to
    stay out of it."""
    plan = network.optimise(synth.make_config(3)[0])
    m, other = (build_host_model(plan, 1 << 20)[0] for _ in range(2))
    for model in (m, other):
        model.fuse_blocks(True)
    done = threading.Event()

    def turn():
        while not done.is_set():
            for switch in ("bottleneck_fuse", "conv1x1_fuse"):
                B.fupr_tuning_set(switch, 0)
                B.fupr_tuning_set(switch, None)

    batches = range(1, 200)
    t = threading.Thread(target=turn)
    t.start()
    try:
        for n in batches:
            for _ in range(20):
                m.num_launches_at(n)
    finally:
        done.set()
        t.join()
        for switch in ("bottleneck_fuse", "conv1x1_fuse"):
            B.fupr_tuning_set(switch, None)
    for n in batches:
        assert m.num_launches_at(n) == other.num_launches_at(n), n


def test_weights_of_2_gib_and_more_stay_out_of_blocks():
    """The kernels of whole blocks read weights through 32-bit offsets, whatever tile is forced."""
    def in_blocks(switch, tile, specs):
        m = B.Model(B.BF16, (16, 2, 2), fake_ops(specs), None)
        m.fuse_blocks(True)
        B.fupr_tuning_set(switch, tile)
        try:
            launches = [m.launch_stats(1, i) for i in range(m.num_launches_at(1))]
            return sum(s["n_ops"] for s in launches if s["kernel"].startswith(("basic_block_", "bottleneck_")))
        finally:
            B.fupr_tuning_set(switch, None)

    def basic(k2):
        return in_blocks("basic_tile", "0x8", [(B.OP_CONV, 0, -1, 16, 16, 3, 1, 1, B.FUSE_RELU, 1),
                                               (B.OP_CONV, 1, -1, k2, 16, 3, 1, 1, B.FUSE_RELU, 1),
                                               (B.OP_AVGPOOL, 2, -1, 1, 1, 1, 1, 0, 0, 1)])

    def bottleneck(k1, k2, k3):
        add = B.FUSE_RELU | B.FUSE_ADD       # (three tensors side by side: buffers for the block's)
        return in_blocks("bottleneck_tile", 0, [(B.OP_CONV, 0, -1, 16, 16, 1, 1, 0, B.FUSE_RELU, 1),
                                                (B.OP_CONV, 1, -1, 16, 16, 1, 1, 0, B.FUSE_RELU, 1),
                                                (B.OP_CONV, 1, 2, 16, 16, 1, 1, 0, add, 1),
                                                (B.OP_CONV, 3, -1, k1, 16, 3, 1, 1, B.FUSE_RELU, 1),
                                                (B.OP_CONV, 4, -1, k2, k1, 1, 1, 0, B.FUSE_RELU, 1),
                                                (B.OP_CONV, 5, -1, k3, k2, 1, 1, 0, B.FUSE_RELU, 1),
                                                (B.OP_AVGPOOL, 6, -1, 1, 1, 1, 1, 0, 0, 1)])

    # 20 chunks of 16 bytes per filter of the second 3 x 3: 2 GiB at 6.7 million, 4 GiB at 13.4 million
    for k2, takes in [(6 << 20, 2), (7 << 20, 0), (14 << 20, 0)]:
        assert basic(k2) == takes, k2
    # 64 bytes per filter of the second; 2 per filter of the third and channel, which can stay outside
    for k2, k3, takes in [(1 << 20, 16, 3), (31 << 20, 16, 3), (33 << 20, 16, 0), (65 << 20, 16, 0),
                          (8 << 20, 112, 3), (8 << 20, 128, 2)]:
        assert bottleneck(16, k2, k3) == takes, (k2, k3)


@pytest.mark.parametrize("config,switch", [(3, "bottleneck_fuse"), (2, "basic_fuse")])
def test_a_launch_list_is_worked_out_once(config, switch):
    """Switches may change while a list is looked at: what a launch is, which plan it has and what it does
    come from one look."""
    m, _ = build_host_model(network.optimise(synth.make_config(config)[0]), 1 << 20)
    m.fuse_blocks(True)
    block = {2: "basic_block_", 3: "bottleneck_"}[config]
    done = threading.Event()

    def turn():
        while not done.is_set():
            B.fupr_tuning_set(switch, 0)
            B.fupr_tuning_set(switch, None)

    t = threading.Thread(target=turn)
    t.start()
    try:
        seen = set()
        for k in range(400 * m.num_ops):
            if k >= 10 * m.num_ops and len(seen) == 2:
                break
            i = k % m.num_ops
            out = B.OpStats()
            st = B._lib.fupr_model_launch_stats(m._h, 64, i, B.C.byref(out))
            assert st in (B.FUPR_OK, B.ERR_ARG)        # (one list is shorter than the other)
            if st == B.FUPR_OK:
                name = out.kernel.decode()
                seen.add(name.startswith(block))
                assert name.startswith(block) or out.n_ops <= 2 and not name.startswith("none"), (i, name, out.n_ops)
        assert seen == {True, False}
    finally:
        done.set()
        t.join()
        B.fupr_tuning_set(switch, None)


# ---- a block's pruned output filters (Alg. 1 on every non-fused operator, Sec. V-A) ---------

def scatter_ops(keep=0x2000, **change):
    """stem, conv1, conv2 whose 11 kept filters add into the stem's 16 channels, head."""
    specs = [
        (B.OP_CONV, 0, -1, 16, 3, 3, 1, 1, B.FUSE_RELU, 1),                          # t1 16 x 32 x 32
        (B.OP_CONV, 1, -1, 10, 16, 3, 1, 1, B.FUSE_RELU, 1),                         # t2
        (B.OP_CONV, 2, 1, 11, 10, 3, 1, 1, B.FUSE_RELU | B.FUSE_ADD | B.FUSE_SCATTER, 1),  # t3 = t1 updated
        (B.OP_AVGPOOL, 3, -1, 1, 1, 1, 1, 0, 0, 1),
        (B.OP_CONV, 4, -1, 10, 16, 1, 1, 0, 0, 1),
    ]
    for i, spec in change.get("specs", {}).items():
        specs[i] = spec
    ops = fake_ops(specs)
    ops[2].keep_idx = keep
    return ops


def test_model_plan_updates_the_stream_in_place():
    m = B.Model(B.BF16, (3, 32, 32), scatter_ops(), None)
    # t1 and t2 only: the update needs no buffer of its own
    assert m.workspace_bytes(1) == 2 * 32 * 32 * 16 * 2
    s = m.op_stats(2, 2)
    assert s["K"] == 11 and s["C"] == 10
    assert s["flops"] == 2.0 * 10 * 9 * 11 * 2 * 1024
    # input once, 11 channels of the stream read and written, parameters, index list
    assert s["bytes"] == 2 * (2 * 1024 * 10 + 2 * 2 * 1024 * 11 + 11 * 10 * 9) + 8 * 11
    assert s["kernel"].startswith("conv3x3p_") or s["kernel"].startswith("conv16t_")
    t = m.output_shape(3)
    assert (t.C, t.c_stride) == (10, 16)
    # no one-kernel schedule with such an operator
    assert m.num_launches == m.num_ops


def test_model_create_errors_of_in_place_updates():
    S = B.FUSE_RELU | B.FUSE_ADD | B.FUSE_SCATTER
    expect(B.ERR_NULL, lambda: B.Model(B.BF16, (3, 32, 32), scatter_ops(keep=None), None))
    cases = [
        ({2: (B.OP_CONV, 2, -1, 11, 10, 3, 1, 1, B.FUSE_RELU | B.FUSE_SCATTER, 1)}, B.ERR_ARG),  # no tensor
        ({2: (B.OP_CONV, 2, 1, 17, 10, 3, 1, 1, S, 1)}, B.ERR_SHAPE),          # more filters than channels
        ({2: (B.OP_CONV, 2, 1, 11, 10, 3, 2, 1, S, 1)}, B.ERR_SHAPE),          # other extent
        ({2: (B.OP_CONV, 2, 1, 11, 10, 3, 1, 1, S, 2)}, B.ERR_ARG),            # strided shortcut
        ({1: (B.OP_CONV, 0, -1, 10, 3, 3, 1, 1, B.FUSE_RELU, 1),
          2: (B.OP_CONV, 2, 0, 3, 10, 3, 1, 1, S, 1)}, B.ERR_ARG),             # the network input
        ({3: (B.OP_CONV, 1, -1, 10, 16, 1, 1, 0, 0, 1),
          4: (B.OP_CONV, 3, -1, 10, 16, 1, 1, 0, 0, 1)}, B.ERR_ARG),           # old number read later
    ]
    for change, code in cases:
        expect(code, lambda: B.Model(B.BF16, (3, 32, 32), scatter_ops(specs=change), None))
    expect(B.ERR_DTYPE, lambda: B.Model(B.F32, (3, 32, 32), scatter_ops(), None))
    last = scatter_ops()[:3]
    expect(B.ERR_ARG, lambda: B.Model(B.BF16, (3, 32, 32), last, None))       # the network's last operator
    plain = fake_ops([(B.OP_CONV, 0, -1, 16, 3, 3, 1, 1, B.FUSE_RELU, 1)])
    plain[0].keep_idx = 0x2000
    expect(B.ERR_ARG, lambda: B.Model(B.BF16, (3, 32, 32), plain, None))      # index list without the flag


def test_output_filter_plan_matches_oracle():
    """Masks and kept-filter lists of the blocks' last convolutions are the oracle's,
    the compacted weights are its extraction, and only identity blocks take part."""
    model = synth.make_imagenet_basic_resnet(23, "bf16", (2, 1, 2, 1), 300, widths=(4, 8, 8, 12),
                                             size=32, classes=7, out_permille=500)
    plan = network.optimise(model)
    masks = orc.select_masks(model)
    assert set(plan["masks"]) == set(masks)
    thin = orc.extract(model, masks)
    by_site = {L.site: L for L in plan["layers"]}
    n_stream = 0
    for bi, blk in enumerate(thin["blocks"]):
        L = by_site[f"b{bi}.conv2"]
        if "stream_keep" in blk:
            assert blk["shortcut"]["kind"] == "identity"
            assert np.array_equal(L.keep, blk["stream_keep"]) and L.keep.dtype == np.int32
            assert np.array_equal(plan["masks"][(bi, 1)], masks[(bi, 1)])
            n_stream += 1
        else:
            assert L.keep is None
        wo, bo = orc.fold(blk["convs"][1]["W"], blk["bns"][1])
        assert L.W.shape == wo.shape
        np.testing.assert_allclose(L.W, wo, rtol=2 ** -23)
        np.testing.assert_allclose(L.bias, bo, rtol=2 ** -22, atol=1e-9)
    assert n_stream == 3
    proj = synth.make_imagenet_basic_resnet(26, "bf16", (1, 1), 300, widths=(4, 8), size=16, classes=3)
    proj["blocks"][1]["prune_permille"][1] = 300
    with pytest.raises(ValueError):
        network.optimise(proj)


# ---- aggressive fusion (Sec. IV-B) -------------------------------------------------

def fusible_blocks():
    a = synth.make_cifar_resnet(21, "bf16", 2, 400, widths=(4, 8, 12), size=12, classes=5)
    b = synth.make_imagenet_basic_resnet(22, "bf16", (1, 2, 1, 1), 300, widths=(4, 8, 8, 12), size=32,
                                         classes=7)
    return a["blocks"] + b["blocks"]


def test_xconv_fuse_matches_oracle_construction():
    kinds = set()
    for blk in fusible_blocks():
        kinds.add(blk["shortcut"]["kind"])
        got = network._aggressive(blk)
        ref = orc.aggressive_fuse_block(blk)
        for ci in range(2):
            a, b = got["convs"][ci]["W"], ref["convs"][ci]["W"]
            assert a.dtype == np.float32 and a.shape == b.shape
            np.testing.assert_allclose(a, b, rtol=2e-7, atol=0)
            assert np.array_equal(a == 0, b == 0)
            for key in ("gamma", "beta", "mean", "var"):
                np.testing.assert_allclose(got["bns"][ci][key], ref["bns"][ci][key], rtol=2e-7, atol=1e-9)
        n, m = got["convs"][0]["W"].shape[0], ref["original_filters"][0]
        assert got["prune_counts"] == [n - m, 0]
    assert kinds == {"identity", "optionA", "projection"}


def test_aggressive_plan_selects_the_oracles_filters():
    model = synth.make_imagenet_basic_resnet(22, "bf16", (1, 2, 1, 1), 300, widths=(4, 8, 8, 12),
                                             size=32, classes=7)
    plan = network.optimise(model, aggressive=True)
    masks = orc.select_masks(orc.aggressive_fuse(model))
    assert set(plan["masks"]) == set(masks)
    for key in masks:
        assert np.array_equal(plan["masks"][key], masks[key])
    assert not any(L.add for L in plan["layers"])
    unpruned = network.optimise(model, aggressive=True, prune_fused=False)
    assert not unpruned["masks"]
    k, c = model["blocks"][0]["convs"][0]["W"].shape[:2]
    by_site = {L.site: L for L in unpruned["layers"]}
    assert by_site["b0.conv1"].W.shape == (k + c, c, 3, 3)
    assert by_site["b0.conv2"].W.shape == (k, k + c, 3, 3)


def test_partially_fused_plan_selects_the_oracles_filters():
    """Fusion option x/n: the blocks of the first x stages go through fupr_xconv_fuse
    and lose n - m filters, the rest are pruned at their rate; masks equal the oracle's."""
    model = synth.make_imagenet_basic_resnet(23, "bf16", (1, 2, 1, 1), 300, widths=(4, 8, 8, 12),
                                             size=32, classes=7)
    for stages in (0, 1, 3, 4):
        plan = network.optimise(model, aggressive=True, fuse_stages=stages)
        masks = orc.select_masks(orc.aggressive_fuse(model, stages=stages))
        assert set(plan["masks"]) == set(masks)
        for key in masks:
            assert np.array_equal(plan["masks"][key], masks[key])
        fused = sum(b["stage"] < stages for b in model["blocks"])
        assert sum(L.add for L in plan["layers"]) == len(model["blocks"]) - fused


def test_proj_concat_is_the_filterwise_concatenation():
    """conv(h, W) + conv_p(x, Wp) = conv([h ; x], [W | Wp]) (Sec. IV-B-1): exact copies of
    both weight sets with zeros between them up to a multiple of 64 channels, biases added;
    the oracle's two convolutions and addition equal its one convolution of the concatenation."""
    rng = np.random.default_rng(12)
    k, c1, c2 = 20, 20, 24
    assert B.CAT_ALIGN == 64
    W = rng.standard_normal((k, c1, 1, 1)).astype(np.float32)
    Wp = rng.standard_normal((k, c2, 1, 1)).astype(np.float32)
    b, bp = rng.standard_normal(k).astype(np.float32), rng.standard_normal(k).astype(np.float32)
    sh, shp = B.shape_of(W, 1, 0), B.shape_of(Wp, 2, 0)
    out, Wc, bc = B.fupr_proj_concat(sh, W, b, shp, Wp, bp)
    assert (out.K, out.C, out.R, out.S, out.stride, out.pad) == (k, 64 + c2, 1, 1, 1, 0)
    assert np.array_equal(Wc[:, :c1], W) and not Wc[:, c1:64].any() and np.array_equal(Wc[:, 64:], Wp)
    assert np.array_equal(bc, b + bp)
    h = rng.standard_normal((2, c1, 5, 6))
    x = rng.standard_normal((2, c2, 10, 12))
    two = orc.add(orc.conv2d(h, W, 1, 0), orc.conv2d(x, Wp, 2, 0))
    cat = np.concatenate([h, np.zeros((2, 64 - c1, 5, 6)), x[:, :, ::2, ::2]], axis=1)
    one = orc.conv2d(cat, Wc, 1, 0)
    np.testing.assert_allclose(one, two, rtol=1e-12, atol=1e-12)
    # errors: a 3 x 3 last convolution, different filter counts, a strided last convolution
    W3 = np.zeros((k, c1, 3, 3), np.float32)
    for bad_last, bad_proj in ((B.shape_of(W3, 1, 1), shp), (sh, B.conv_shape(k + 1, c2, 1, 1, 2, 0)),
                               (B.conv_shape(k, c1, 1, 1, 2, 0), shp)):
        with pytest.raises(B.FuprError) as e:
            B.fupr_proj_concat(bad_last, W3 if bad_last.R == 3 else W, b, bad_proj,
                               np.zeros((bad_proj.K, c2, 1, 1), np.float32), None)
        assert e.value.status == B.ERR_SHAPE


def test_model_accepts_a_two_input_convolution():
    def ops(in2=1, stride=2, c=64 + 16, epi=B.FUSE_RELU | B.FUSE_CAT):
        o = fake_ops([
            (B.OP_CONV, 0, -1, 16, 3, 3, 1, 1, B.FUSE_RELU, 1),      # t1 16 x 32 x 32
            (B.OP_CONV, 1, -1, 12, 16, 3, 2, 1, B.FUSE_RELU, 1),     # t2 12 x 16 x 16
            (B.OP_CONV, 2, -1, 40, c, 1, 1, 0, epi, 1),              # t3 = conv([t2 ; t1 at stride 2])
        ])
        o[2].in2, o[2].in2_spatial_stride = in2, stride
        return o
    m = B.Model(B.BF16, (3, 32, 32), ops(), None)
    s = m.op_stats(2, 2)
    assert s["flops"] == 2.0 * (12 + 16) * 40 * 2 * 256 and s["C"] == 28
    # t1 stays alive until the last operator: three buffers... t1 and t2 only (t3 is the output)
    assert m.workspace_bytes(1) == (32 * 32 * 16 + 16 * 16 * 16) * 2
    expect(B.ERR_SHAPE, lambda: B.Model(B.BF16, (3, 32, 32), ops(c=32 + 16), None))   # split not at 64
    expect(B.ERR_ARG, lambda: B.Model(B.BF16, (3, 32, 32), ops(in2=3), None))
    expect(B.ERR_ARG, lambda: B.Model(B.BF16, (3, 32, 32), ops(stride=3), None))
    B.Model(B.BF16, (3, 32, 32), ops(in2=0, c=64 + 3, stride=1), None)      # any earlier tensor large enough
    expect(B.ERR_SHAPE, lambda: B.Model(B.BF16, (3, 32, 32), ops(in2=2, c=64 + 12, stride=2), None))  # too small
    expect(B.ERR_DTYPE, lambda: B.Model(B.F32, (3, 32, 32), ops(), None))


def test_xconv_fuse_errors():
    blk = fusible_blocks()[0]
    c1, c2 = blk["convs"]
    b1, b2 = blk["bns"]
    # a zero scale after conv2 cannot be inverted
    bad = dict(b2)
    g = b2["gamma"].copy()
    g[1] = 0.0
    bad["gamma"] = g
    with pytest.raises(B.FuprError) as e:
        B.fupr_xconv_fuse(c1, b1, c2, bad, B.SHORTCUT_IDENTITY)
    assert e.value.status == B.ERR_BN_SCALE
    # var + eps must be positive
    bad = dict(b2)
    bad["var"] = -np.ones_like(b2["var"])
    with pytest.raises(B.FuprError) as e:
        B.fupr_xconv_fuse(c1, b1, c2, bad, B.SHORTCUT_IDENTITY)
    assert e.value.status == B.ERR_BN_VAR
    # unknown shortcut kind, projection without its convolution, mismatched conv2
    with pytest.raises(B.FuprError) as e:
        B.fupr_xconv_fuse(c1, b1, c2, b2, 7)
    assert e.value.status == B.ERR_ARG
    with pytest.raises(B.FuprError) as e:
        B.fupr_xconv_fuse(c1, b1, c2, b2, B.SHORTCUT_PROJECTION)
    assert e.value.status == B.ERR_NULL
    wrong = {"W": np.zeros((4, 5, 3, 3), np.float32), "stride": 1, "pad": 1}
    with pytest.raises(B.FuprError) as e:
        B.fupr_xconv_fuse(c1, b1, wrong, b2, B.SHORTCUT_IDENTITY)
    assert e.value.status == B.ERR_SHAPE
    even = {"W": np.zeros((4, 4, 2, 2), np.float32), "stride": 1, "pad": 1}
    with pytest.raises(B.FuprError) as e:
        B.fupr_xconv_fuse(even, b1, even, b2, B.SHORTCUT_IDENTITY)
    assert e.value.status == B.ERR_SHAPE


def test_bench_refuses_more_than_one_gpu():
    """The benchmark measures one GPU; asking for more must end with a message, not a run."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in r.stderr
