"""GPU parity of the channels-last execution (matrix-core convolutions over [row][column][channel]
tensors) on small nets chosen for its edges: tiles that are not full, channel counts that are not
whole K steps, first layers of few channels, strides, residuals, fused projections, in-place and copied
concatenations, flat outputs, every tile and K split.  Buffers and outputs against the oracle with the
propagated bound of a forward error analysis (util.chain_bounds)."""
import re

import numpy as np
import pytest

import oracle
import workloads as wl
from util import chain_bounds, assert_within_bound

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

Op = wl.Op


@pytest.fixture(scope="module")
def cad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1905_00571_amd as cad
    cad.lib()
    return cad


def stem_net():
    """7x7/2 first layer on 3 channels, max pool, depthwise, a strided block with projection, an
    identity block, a concatenation with one in-place, one pooled and one copied source, a fully
    connected layer on a map of several pixels."""
    return [
        Op("conv", "stem", 0, 1, 3, 24, 7, 2, 3, 0.0, True),
        Op("maxpool", "pool", 1, 2, k=3, stride=2, pad=1),
        Op("conv", "expand", 2, 3, 24, 72, 1, 1, 0, 0.5, True),
        Op("dwconv", "dw1", 3, 4, 72, 72, 3, 1, 1, 0.0, True),
        Op("conv", "project", 4, 5, 72, 40, 1, 1, 0, 0.5, False),
        Op("conv", "a", 5, 6, 40, 16, 1, 1, 0, 0.5, True),
        Op("conv", "b", 6, 7, 16, 16, 3, 2, 1, 0.5, True),
        Op("conv", "p", 5, 8, 40, 136, 1, 2, 0, 0.5, False),
        Op("conv", "c", 7, 9, 16, 136, 1, 1, 0, 0.5, True, 8),
        Op("dwconv", "dw2", 9, 10, 136, 136, 3, 2, 1, 0.0, False),
        Op("conv", "d", 10, 11, 136, 64, 3, 1, 1, 0.8, True),
        Op("conv", "e", 11, 12, 64, 64, 3, 1, 1, 0.8, True, 11),
        Op("avgpool2d", "mean", 12, 13, k=3, stride=1, pad=1),
        Op("conv", "f", 13, 14, 64, 24, 1, 1, 0, 0.5, True),
        Op("concat", "cat", 12, 15, srcs=(12, 14)),
        Op("maxpool", "last", 15, 16, k=2, stride=1, pad=0),
        Op("fc", "fc", 16, 17, 88 * 2 * 3, 30, sparsity=0.5, relu=False),
    ], (3, 3, 43, 51)


def deep_net():
    """An input of many channels (brought in by a transposition, read as a residual too), a long K on few
    pixels (K splits), a rectangular filter in a square bank, an output that is a feature map."""
    return [
        Op("conv", "in", 0, 1, 264, 72, 1, 1, 0, 0.8, True),
        Op("conv", "long", 1, 2, 72, 200, 3, 1, 1, 0.8, True),
        Op("conv", "rect", 2, 3, 200, 136, 7, 1, 3, 0.5, True, kh=1, kw=7),
        Op("conv", "back", 3, 4, 136, 264, 1, 1, 0, 0.8, False, 0),
        Op("conv", "out", 4, 5, 264, 72, 5, 2, 2, 0.9, True),
    ], (5, 264, 6, 5)


def mean_net():
    """A 3x3 first layer, one image, the global average pool in front of the classifier."""
    return [
        Op("conv", "stem", 0, 1, 3, 8, 3, 2, 1, 0.0, True),
        Op("conv", "wide", 1, 2, 8, 136, 3, 2, 0, 0.5, True),
        Op("avgpool", "gap", 2, 3),
        Op("fc", "fc", 3, 4, 136, 12, sparsity=0.5, relu=True),
    ], (1, 3, 20, 23)


@pytest.mark.parametrize("dtype_name", ["f32", "f16"])
@pytest.mark.parametrize("make", [stem_net, deep_net, mean_net], ids=lambda f: f.__name__)
def test_channels_last_net(cad, make, dtype_name):
    f16 = dtype_name == "f16"
    dtype, npdt = (cad.F16, np.float16) if f16 else (cad.F32, np.float32)
    ops, shape = make()
    x, ws, bs = wl.net_tensors(ops, make.__name__, shape, input_relu=True)
    xs = x.astype(npdt)
    ref, ins, outs = oracle.run_net(ops, xs, ws, bs, dtype=npdt)
    bounds = chain_bounds(ops, ins, outs, ws, bs, f16)
    xs2 = wl.activation(shape, make.__name__, 99, relu=True).astype(npdt)
    ref2, ins2, outs2 = oracle.run_net(ops, xs2, ws, bs, dtype=npdt)
    bound2 = chain_bounds(ops, ins2, outs2, ws, bs, f16)[-1]

    net = cad.build_net(ops, ws, bs, shape, dtype, use_graph=True)
    planes = net.variants()
    convs = [i for i, o in enumerate(ops) if o.kind == "conv"]
    net.set_op_variant(convs[0], "cl_mfma_64x64_s3")          # the whole net goes channels-last

    def check(what):
        for inp, want, lim in ((xs, ref, bounds[-1]), (xs2, ref2, bound2), (xs, ref, bounds[-1])):
            y = net.run(torch.from_numpy(inp).cuda())
            torch.cuda.synchronize()
            assert_within_bound(y.cpu().numpy(), want, lim, f"{make.__name__} {what}")
        checked = 0
        for i, o in enumerate(ops[:-1]):
            if net.op_variant(i) == "fused":
                with pytest.raises(cad.CadnnError):
                    net.read_buffer(o.dst, outs[i].shape)
                continue
            assert_within_bound(net.read_buffer(o.dst, outs[i].shape), outs[i], bounds[i], f"{make.__name__} {what} {o.name}")
            checked += 1
        return checked

    check("default tiles")
    names = {i: net.op_candidates(i) for i in convs if net.op_variant(i) != "fused"}
    every = sorted(set(sum(names.values(), [])))
    for name in every:
        for i, have in names.items():
            net.set_op_variant(i, name if name in have else None)
            assert name not in have or net.op_variant(i) == name
        check(name)
    if make is deep_net:
        assert {"cl_mfma_128x128_s2", "cl_mfma_64x64_s3k4", "cl_mfma_64x64_s4k4"} <= set(every), every
    with pytest.raises(cad.CadnnError):
        net.set_op_variant(convs[0], "cl_no_such_tile")
    saved = net.variants()
    net.set_variants(planes)                                # and back
    assert net.variants() == planes
    y = net.run(torch.from_numpy(xs).cuda())
    torch.cuda.synchronize()
    assert_within_bound(y.cpu().numpy(), ref, bounds[-1], f"{make.__name__} back on planes")
    net.set_variants(saved)
    assert net.variants() == saved
    check("saved choice replayed")
    net.free()


def test_channels_last_tuned(cad):
    """A net the rule takes channels-last by itself (enough multiply-adds), tuned on its first run."""
    ops = wl.resnet50_ops(uniform=0.8)
    shape = (8, 3, 128, 127)
    x, ws, bs = wl.net_tensors(ops, "cl-tuned", shape)
    xs = x.astype(np.float16)
    ref, _, _ = oracle.run_net(ops, xs, ws, bs, dtype=np.float16)
    net = cad.build_net(ops, ws, bs, shape, cad.F16, use_graph=True, tune=True)
    for _ in range(2):
        y = net.run(torch.from_numpy(xs).cuda())
        torch.cuda.synchronize()
        got = y.float().cpu().numpy()
        # 1e-2: the stated bar of whole nets in fp16 storage
        assert np.abs(got - ref).max() <= 1e-2 * np.abs(ref).max()
    assert all(n.startswith("cl_") or n == "fused" for n, o in zip(net.variants(), ops) if o.kind == "conv")
    net.free()


def test_tuning_in_2_byte_storage_leaves_out_two_wave_groups(cad, capfd, monkeypatch):
    """They win a layer timed alone, which is what tuning measures, and lose the net: offered for a pin, never tuned to."""
    ops = [Op("conv", f"c{i}", i, i + 1, 256, 256, 3, 1, 1, 0.8, True) for i in range(2)]
    x, ws, bs = wl.net_tensors(ops, "tune-groups", (2, 256, 14, 14))
    monkeypatch.setenv("CADNN_TUNE_LOG", "1")
    for dtype, tuned in ((cad.F16, False), (cad.F32, True)):
        net = cad.build_net(ops, ws, bs, x.shape, dtype, use_graph=False, tune=True)
        net.set_op_variant(0, "cl_mfma_64x64_s3")
        xd = torch.from_numpy(x).cuda()
        net.run(xd.half() if dtype == cad.F16 else xd)
        torch.cuda.synchronize()
        names = net.op_candidates(0)
        assert "cl_mfma_64x64_s3g2" in names
        timed = [line for line in capfd.readouterr().err.splitlines() if line.startswith("[cadnn tune] cl ")]
        assert timed and any("s3g2" in line for line in timed) == tuned
        net.set_op_variant(0, "cl_mfma_64x64_s3g2")
        assert net.op_variant(0) == "cl_mfma_64x64_s3g2"
        net.free()


@pytest.mark.parametrize("family,shape", [("mobilenet_v1", (16, 3, 128, 129)), ("vgg16", (2, 3, 96, 112))])
def test_tuning_times_both_executions(cad, family, shape, capfd, monkeypatch):
    """A net that the rule takes channels-last is tuned on plane layouts too, and what stays is the execution whose
    whole pass was the faster one; either computes the net, run after run, with what tuning left in the workspace."""
    ops = wl.mobilenet_v1_ops() if family == "mobilenet_v1" else wl.vgg16_ops()[:-3]
    if family == "vgg16":
        ops.append(Op("avgpool", "gap", ops[-1].dst, 9))
    x, ws, bs = wl.net_tensors(ops, "both", shape)
    xs = x.astype(np.float16)
    ref, _, _ = oracle.run_net(ops, xs, ws, bs, dtype=np.float16)
    monkeypatch.setenv("CADNN_TUNE_LOG", "1")
    plain = cad.build_net(ops, ws, bs, shape, cad.F16, use_graph=True)
    first = next(i for i, o in enumerate(ops) if o.kind == "conv")
    by_rule = plain.op_variant(first).startswith("cl_")
    plain.free()
    assert by_rule
    net = cad.build_net(ops, ws, bs, shape, cad.F16, use_graph=True, tune=True)
    for _ in range(3):
        y = net.run(torch.from_numpy(xs).cuda())
        torch.cuda.synchronize()
        assert np.abs(y.float().cpu().numpy() - ref).max() <= 1e-2 * np.abs(ref).max()      # (whole nets in fp16 storage)
    log = capfd.readouterr().err
    assert "[cadnn tune] cl " in log and "[cadnn tune] cin=" in log
    m = re.search(r"whole pass: channels-last ([\d.]+) us, planes ([\d.]+) us", log)
    assert net.op_variant(first).startswith("cl_") == (float(m[1]) <= float(m[2]))
    net.free()


@pytest.mark.parametrize("dtype_name", ["f32", "f16"])
@pytest.mark.parametrize("k,stride,pad,h,w", [(3, 2, 0, 19, 23), (3, 1, 1, 9, 14), (7, 2, 3, 21, 20), (7, 2, 0, 15, 17), (5, 1, 0, 11, 9),
                                              (5, 2, 2, 12, 13), (4, 2, 1, 12, 14), (1, 1, 0, 6, 7), (2, 2, 0, 10, 12)])
def test_first_layer_reads_nothing_outside_its_windows(cad, k, stride, pad, h, w, dtype_name):
    """A packed first layer's K step is wider than a filter row.  NaN and infinities in the middle image, at its
    corners, edges and inside: every output whose window holds none of them (all of the other images') has the
    bits it has without them, with every tile."""
    dtype, npdt = (cad.F16, np.float16) if dtype_name == "f16" else (cad.F32, np.float32)
    ops = [Op("conv", "stem", 0, 1, 3, 40, k, stride, pad, 0.0, False), Op("conv", "next", 1, 2, 40, 8, 1, 1, 0, 0.5, False)]
    shape = (3, 3, h, w)
    x, ws, bs = wl.net_tensors(ops, f"stem-{k}-{stride}-{pad}", shape)
    bad = x.astype(npdt)
    hit = np.zeros((3, h, w), bool)
    for i, (r, c) in enumerate([(0, 0), (0, w - 1), (h - 1, 0), (h - 1, w - 1), (h // 2, 0), (h // 2, w // 2), (h // 2, w - 1)]):
        bad[1, i % 3, r, c] = (np.nan, np.inf, -np.inf)[i % 3]
        hit[1, r, c] = True
    ho, wo = wl.conv_out_size(h, k, stride, pad), wl.conv_out_size(w, k, stride, pad)
    padded = np.pad(hit, ((0, 0), (pad, pad + k), (pad, pad + k)))
    touched = np.zeros((3, ho, wo), bool)
    for a in range(k):
        for b in range(k):
            touched |= padded[:, a:a + ho * stride:stride, b:b + wo * stride:stride][:, :ho, :wo]
    assert touched[1].any() and not touched[1].all()
    net = cad.build_net(ops, ws, bs, shape, dtype, use_graph=False)
    net.set_op_variant(0, "cl_mfma_64x64_s3")
    keep = np.broadcast_to(~touched[:, None], (3, 40, ho, wo))
    for name in net.op_candidates(0):
        net.set_op_variant(0, name)
        maps = []
        for inp in (x.astype(npdt), bad):
            net.run(torch.from_numpy(inp).cuda())
            torch.cuda.synchronize()
            maps.append(net.read_buffer(1, (3, 40, ho, wo)))
        assert np.isfinite(maps[0]).all() and not np.isfinite(maps[1]).all()
        assert np.array_equal(maps[0][keep], maps[1][keep]), name
    net.free()


@pytest.mark.parametrize("n,cin,cout,k,stride,h,w", [(1, 8, 8, 1, 1, 3, 5),          # one step: seven waves have nothing of K
                                                     (1, 40, 24, 3, 1, 4, 4),         # rows of 64 bytes, one whole block of pixels
                                                     (2, 96, 72, 3, 2, 9, 7),         # an odd number of half steps, pixels across images
                                                     (1, 64, 136, 1, 1, 17, 1),       # a pixel more than a block
                                                     (3, 160, 40, 5, 1, 6, 6),        # parts of K that end inside a tap
                                                     (1, 520, 16, 3, 1, 7, 7)])
def test_small_tiles(cad, n, cin, cout, k, stride, h, w):
    """The variants whose waves share K, at the ends of their tiles and of K, with a residual and a fused projection: within
    fp32 sums of K products and one rounding to fp16 of 64-bit arithmetic."""
    ops = [Op("conv", "in", 0, 1, cin, cin, 1, 1, 0, 0.0, False), Op("conv", "p", 1, 2, cin, cout, 1, stride, 0, 0.0, False),
           Op("conv", "a", 1, 3, cin, cout, k, stride, k // 2, 0.0, True, 2), Op("conv", "b", 3, 4, cout, cout, 1, 1, 0, 0.0, True, 3),
           Op("conv", "out", 4, 5, cout, 8, 1, 1, 0, 0.5, False)]
    x, ws, bs = wl.net_tensors(ops, "small", (n, cin, h, w))
    x = x.astype(np.float16)
    net = cad.build_net(ops, ws, bs, x.shape, cad.F16, use_graph=False)
    net.set_op_variant(0, "cl_mfma_64x64_s3")
    names = [v for v in net.op_candidates(2) if v.endswith("_w8")]
    assert len(names) == 4
    conv = torch.nn.functional.conv2d

    def layer(i, t):
        wt = torch.from_numpy(ws[i].astype(np.float16)).double().reshape(ops[i].cout, ops[i].cin, ops[i].k, ops[i].k)
        both = [conv(a, b, c, ops[i].stride, ops[i].pad) for a, b, c in
                ((t, wt, torch.from_numpy(bs[i]).double()), (t.abs(), wt.abs(), torch.from_numpy(np.abs(bs[i])).double()))]
        return both[0].numpy(), both[1].numpy(), ops[i].cin * ops[i].k ** 2

    def check(got, ref, size, terms, what):
        bound = (terms + 3) * 2.0 ** -24 * size + 2.0 ** -11 * np.abs(ref) + 2.0 ** -25
        excess = (np.abs(got.astype(np.float64) - ref) - bound).max()
        assert excess <= 0.0, f"{what}: {excess:.3e} above the bound"

    for name in names:
        for op in (0, 2, 3):
            net.set_op_variant(op, name)
        net.run(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        assert net.op_variant(1) == "fused" and net.op_variant(2) == name
        ho, wo = (wl.conv_out_size(s, k, stride, k // 2) for s in (h, w))
        mid = net.read_buffer(1, (n, cin, h, w))
        a, b = net.read_buffer(3, (n, cout, ho, wo)), net.read_buffer(4, (n, cout, ho, wo))
        ref, size, terms = layer(0, torch.from_numpy(x).double())
        check(mid, ref, size, terms, name + " in")
        (ref, size, terms), (ref2, size2, terms2) = layer(2, torch.from_numpy(mid).double()), layer(1, torch.from_numpy(mid).double())
        check(a, np.maximum(ref + ref2, 0.0), size + size2, terms + terms2, name + " a")
        ref, size, terms = layer(3, torch.from_numpy(a).double())
        r = a.astype(np.float64)
        check(b, np.maximum(ref + r, 0.0), size + np.abs(r), terms, name + " b")
    net.free()


@pytest.mark.parametrize("cin,cout,k", [(32, 128, 3), (16, 256, 3), (160, 128, 1), (352, 256, 1), (480, 128, 1), (416, 384, 1)])
def test_steps_that_the_groups_of_a_split_do_not_share_evenly(cad, cin, cout, k):
    """fp32 storage with every tile, where the last part of K is shorter than the others and the last block of channels ends
    with the weights: what is requested behind the end comes back as zeros.  (K + 3) 2^-24 (sum |w| |x| + |b|)."""
    ops = [Op("conv", "a", 0, 1, cin, cout, k, 1, k // 2, 0.0, False), Op("conv", "b", 1, 2, cout, 8, 1, 1, 0, 0.5, False)]
    x, ws, bs = wl.net_tensors(ops, f"uneven-{cin}-{cout}", (2, cin, 6, 7))
    wt = torch.from_numpy(ws[0]).double().reshape(cout, cin, k, k)
    conv = torch.nn.functional.conv2d
    ref = conv(torch.from_numpy(x).double(), wt, torch.from_numpy(bs[0]).double(), 1, k // 2).numpy()
    size = conv(torch.from_numpy(x).double().abs(), wt.abs(), torch.from_numpy(np.abs(bs[0])).double(), 1, k // 2).numpy()
    net = cad.build_net(ops, ws, bs, x.shape, cad.F32, use_graph=False)
    net.set_op_variant(0, "cl_mfma_64x64_s3")
    names = net.op_candidates(0)
    assert "cl_mfma_64x64_s3g2" in names and "cl_mfma_64x128_s2g2" in names
    for name in names:
        net.set_op_variant(0, name)
        net.run(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        excess = np.abs(net.read_buffer(1, ref.shape).astype(np.float64) - ref) - (cin * k * k + 3) * 2.0 ** -24 * size
        assert excess.max() <= 0.0, f"{name}: {excess.max():.3e} above the bound"
    net.free()


@pytest.mark.parametrize("cin,cout,k,hw", [(8, 40, 3, 9), (64, 136, 1, 13), (96, 72, 3, 10), (160, 264, 3, 6)])
def test_fp32_products_of_extreme_values(cad, cin, cout, k, hw):
    """fp32 storage with every tile: infinities and NaN where 64-bit arithmetic has them (no filter has a zero), and values
    next to the largest and far below one to the accuracy of fp32 sums of K products, (K + 3) 2^-24 (sum |w| |x| + |b|),
    in pixels beside the others as well."""
    rng = np.random.default_rng(cin)
    pad, n = k // 2, 2
    x = rng.standard_normal((n, cin, hw, hw)).astype(np.float32)
    x[0, 1, 0, 0], x[0, cin - 1, 0, hw - 1], x[0, 0, hw - 1, 0] = np.inf, -np.inf, np.nan
    x[1, :, : hw // 2] *= np.float32(1e-30)
    x[1, 3, hw - 1, hw - 1], x[1, 2, hw - 1, 0] = np.finfo(np.float32).max, np.float32(-3.395e38)
    w = (rng.choice([-1.0, 1.0], (cout, cin, k, k)) * rng.uniform(0.1, 1.0, (cout, cin, k, k)) / (cin * k * k)).astype(np.float32)
    b = np.zeros(cout, np.float32)
    ops = [Op("conv", "a", 0, 1, cin, cout, k, 1, pad, 0.0, False), Op("conv", "b", 1, 2, cout, 8, 1, 1, 0, 0.5, False)]
    _, ws, bs = wl.net_tensors(ops, "extreme", x.shape)
    ws[0], bs[0] = w, b
    conv = torch.nn.functional.conv2d
    ref = conv(torch.from_numpy(x).double(), torch.from_numpy(w).double(), None, 1, pad).numpy()
    size = conv(torch.from_numpy(x).double().abs(), torch.from_numpy(w).double().abs(), None, 1, pad).numpy()
    finite = np.isfinite(ref)
    assert not finite.all() and np.isinf(ref).any() and np.isnan(ref).any()
    net = cad.build_net(ops, ws, bs, x.shape, cad.F32, use_graph=False)
    net.set_op_variant(0, "cl_mfma_64x64_s3")
    for name in net.op_candidates(0):
        net.set_op_variant(0, name)
        net.run(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        got = net.read_buffer(1, ref.shape)
        assert np.array_equal(got[~finite], ref[~finite].astype(np.float32), equal_nan=True), name
        excess = (np.abs(got.astype(np.float64) - ref) - (cin * k * k + 3) * 2.0 ** -24 * size)[finite]
        assert excess.max() <= 0.0, f"{name}: {excess.max():.3e} above the bound"
    net.free()


@pytest.mark.parametrize("cin,cout,k,sparsity", [(64, 64, 1, 0.9), (512, 128, 1, 0.9), (256, 64, 3, 0.8), (64, 64, 3, 0.95), (96, 64, 3, 0.0)])
def test_fp32_sums_are_as_exact_as_a_chain_over_the_nonzeros(cad, cin, cout, k, sparsity):
    """fp32 storage with every tile, against 64 bits: no further off (2-norm) than products and sums of the stored weights alone, one
    after the other in fp32, for zeros add no rounding there.  (1.15: the two are random walks of different steps.)"""
    pad, n, hw = k // 2, 1, 12
    ops = [Op("conv", "a", 0, 1, cin, cout, k, 1, pad, sparsity, False), Op("conv", "b", 1, 2, cout, 8, 1, 1, 0, 0.5, False)]
    x, ws, bs = wl.net_tensors(ops, f"exact-{cin}-{k}", (n, cin, hw, hw), input_relu=True)
    bs[0] = np.zeros(cout, np.float32)
    w = ws[0].reshape(cout, cin, k, k)
    padded = np.pad(x, ((0, 0), (0, 0), (pad, pad), (pad, pad)))
    chain, ref = np.zeros((n, cout, hw, hw), np.float32), np.zeros((n, cout, hw, hw))
    for co in range(cout):
        for ci, r, c in np.argwhere(w[co]):
            part = padded[:, ci, r:r + hw, c:c + hw]
            chain[:, co] += w[co, ci, r, c] * part
            ref[:, co] += np.float64(w[co, ci, r, c]) * part.astype(np.float64)
    off = lambda y: float(np.sqrt(((y - ref) ** 2).sum() / (ref ** 2).sum()))
    net = cad.build_net(ops, ws, bs, x.shape, cad.F32, use_graph=False)
    net.set_op_variant(0, "cl_mfma_64x64_s3")
    for name in net.op_candidates(0):
        net.set_op_variant(0, name)
        net.run(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        got = off(net.read_buffer(1, ref.shape))
        assert got <= 1.15 * off(chain), f"{name}: {got:.3e}, a chain {off(chain):.3e}"
    net.free()


def assert_fp32_sums(got, ref, size, terms, what):
    """Infinities and NaN where 64-bit arithmetic has them, else within (terms + 3) 2^-24 size."""
    finite = np.isfinite(ref)
    assert np.array_equal(got[~finite], ref[~finite].astype(np.float32), equal_nan=True), what
    excess = np.abs(got[finite].astype(np.float64) - ref[finite]) - (terms + 3) * 2.0 ** -24 * size[finite]
    assert excess.max() <= 0.0, f"{what}: {excess.max():.3e} above the bound"


@pytest.mark.parametrize("where", ["main", "shortcut"])
@pytest.mark.parametrize("cin,csc,cout,k", [(96, 64, 72, 3), (40, 24, 136, 1), (64, 160, 40, 3)])
def test_repeat_with_fp32_products_across_a_fused_projection(cad, cin, csc, cout, k, where):
    """An infinity in the layer's own input, or in the input of the stride-2 projection that is more of its K: every tile,
    two wave groups and splits that begin inside the projection among them, gives what 64-bit arithmetic gives on the maps."""
    ops = [Op("conv", "m", 0, 1, 8, cin, 1, 1, 0, 0.0, False), Op("conv", "q", 0, 2, 8, csc, 1, 1, 0, 0.0, False),
           Op("conv", "p", 2, 3, csc, cout, 1, 2, 0, 0.0, False), Op("conv", "a", 1, 4, cin, cout, k, 2, k // 2, 0.0, False, 3),
           Op("conv", "out", 4, 5, cout, 8, 1, 1, 0, 0.5, False)]
    n, h, w = 2, 11, 9
    x, ws, bs = wl.net_tensors(ops, f"repeat-{cin}", (n, 8, h, w))
    x, ws = x.copy(), [None if t is None else t.copy() for t in ws]
    x[0, 3, 4, 4], x[1, 3, 0, 0], x[1, 3, h - 1, w - 1] = 1e30, -1e30, 1e30
    for i in (0, 1):
        ws[i][:, 3] = 1e-30
    ws[0 if where == "main" else 1][5, 3] = 1e30           # (that channel of that map overflows)
    net = cad.build_net(ops, ws, bs, x.shape, cad.F32, use_graph=False)
    net.set_op_variant(0, "cl_mfma_64x64_s3")
    names = net.op_candidates(3)
    assert net.op_variant(2) == "fused" and "cl_mfma_64x64_s3g2" in names
    conv = torch.nn.functional.conv2d
    for name in names:
        net.set_op_variant(3, name)
        net.run(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        maps = [net.read_buffer(1, (n, cin, h, w)), net.read_buffer(2, (n, csc, h, w))]
        assert [bool(np.isinf(m).any()) for m in maps] == [where == "main", where == "shortcut"]
        ref, size = 0.0, 0.0
        for m, i in ((maps[0], 3), (maps[1], 2)):
            t, wt, b = torch.from_numpy(m).double(), torch.from_numpy(ws[i]).double(), torch.from_numpy(bs[i]).double()
            wt = wt.reshape(cout, -1, ops[i].k, ops[i].k)
            ref = ref + conv(t, wt, b, 2, ops[i].pad).numpy()
            size = size + conv(t.abs(), wt.abs(), b.abs(), 2, ops[i].pad).numpy()
        assert not np.isfinite(ref).all() and np.isfinite(ref).any()
        assert_fp32_sums(net.read_buffer(4, ref.shape), ref, size, cin * k * k + csc, name)
    net.free()


@pytest.mark.parametrize("k,stride,pad,h,w", [(3, 2, 0, 19, 23), (7, 2, 3, 21, 20), (5, 1, 0, 11, 9)])
def test_repeat_with_fp32_products_in_a_first_layer(cad, k, stride, pad, h, w):
    """... and in a packed first layer, whose steps are wider than its filter rows."""
    ops = [Op("conv", "stem", 0, 1, 3, 40, k, stride, pad, 0.0, False), Op("conv", "next", 1, 2, 40, 8, 1, 1, 0, 0.5, False)]
    x, ws, bs = wl.net_tensors(ops, f"stem-repeat-{k}", (2, 3, h, w))
    x = x.copy()
    x[0, 1, 0, 0], x[0, 2, h - 1, w - 1], x[0, 0, h // 2, 0], x[1, 0, h // 2, w // 2] = np.inf, -np.inf, np.nan, 3e38
    wt = torch.from_numpy(ws[0]).double().reshape(40, 3, k, k)
    conv = torch.nn.functional.conv2d
    ref = conv(torch.from_numpy(x).double(), wt, torch.from_numpy(bs[0]).double(), stride, pad).numpy()
    size = conv(torch.from_numpy(x).double().abs(), wt.abs(), torch.from_numpy(np.abs(bs[0])).double(), stride, pad).numpy()
    ref[np.abs(ref) > np.finfo(np.float32).max] = np.nan
    sure = np.isfinite(ref)
    net = cad.build_net(ops, ws, bs, x.shape, cad.F32, use_graph=False)
    net.set_op_variant(0, "cl_mfma_64x64_s3")
    for name in net.op_candidates(0):
        net.set_op_variant(0, name)
        net.run(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        got = net.read_buffer(1, ref.shape)
        assert not np.isfinite(got[~sure]).any(), name
        assert_fp32_sums(got[sure], ref[sure], size[sure], 3 * k * k, name)
    net.free()


@pytest.mark.parametrize("cin,cout,k", [(16, 40, 3), (64, 72, 1)])
@pytest.mark.parametrize("x_exp,w_exp", [(-120, 100), (-147, 95), (95, -120), (95, -147), (-60, -60), (0, 0)])
def test_fp32_products_of_operands_of_every_magnitude(cad, cin, cout, k, x_exp, w_exp):
    """fp32 storage with every tile: tiny and subnormal activations under large weights, and the other way round, some
    of them among ordinary ones, count with all of their bits: (K + 3) 2^-24 (sum |w| |x| + |b|).  The last
    pixels hold the operands whose product is furthest from that of its leading parts, all of one sign."""
    rng = np.random.default_rng(1000 + cin + x_exp)
    hw, pad, n = 9, k // 2, 2
    x = np.ldexp(rng.standard_normal((n, cin, hw, hw)), x_exp).astype(np.float32)
    w = np.ldexp(rng.choice([-1.0, 1.0], (cout, cin, k, k)) * rng.uniform(0.1, 1.0, (cout, cin, k, k)), w_exp).astype(np.float32)
    if x_exp == -120:
        x[0, :, :4] = np.ldexp(rng.standard_normal((cin, 4, hw)), 0)                # whole rows of ordinary ones
    if x_exp == 0:
        x[1], w[8:] = 1.0 + 2.0 ** -8 - 2.0 ** -17, 1.0 + 2.0 ** -8 - 2.0 ** -17
    if w_exp == -120:
        w[:, : cin // 2] = 0.0
    ops = [Op("conv", "a", 0, 1, cin, cout, k, 1, pad, 0.0, False), Op("conv", "b", 1, 2, cout, 8, 1, 1, 0, 0.5, False)]
    _, ws, bs = wl.net_tensors(ops, "magnitudes", x.shape)
    ws[0], bs[0] = w, np.zeros(cout, np.float32)
    conv = torch.nn.functional.conv2d
    ref = conv(torch.from_numpy(x).double(), torch.from_numpy(w).double(), None, 1, pad)
    size = conv(torch.from_numpy(x).double().abs(), torch.from_numpy(w).double().abs(), None, 1, pad)
    # (a sum that ends below the normal numbers is rounded to a multiple of 2^-149)
    bound = (cin * k * k + 3) * 2.0 ** -24 * size + 2.0 ** -149

    def check(got, what):
        excess = ((torch.as_tensor(got).double().cpu() - ref).abs() - bound).max().item()
        assert excess <= 0.0, f"{what}: {excess:.3e} above the bound"

    net = cad.build_net(ops, ws, bs, x.shape, cad.F32, use_graph=False)
    net.set_op_variant(0, "cl_mfma_64x64_s3")
    for name in net.op_candidates(0):
        net.set_op_variant(0, name)
        net.run(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        check(net.read_buffer(1, tuple(ref.shape)), name)
    net.free()
    check(cad.cadnn_dense_conv2d(torch.from_numpy(w).cuda(), torch.from_numpy(x).cuda(), 1, pad), "layer call")


@pytest.mark.parametrize("dtype_name", ["f32", "f16"])
@pytest.mark.parametrize("k,pad", [(1, 0), (2, 0), (2, 1), (3, 1), (3, 0), (5, 2)])
def test_pools_and_copies_of_non_finite_values(cad, k, pad, dtype_name):
    """Maximum pools over maps with NaN and infinities (whole windows of NaN among them), and the copy of such a
    map into a concatenation, give what the pools on planes give: the window's first element inside the image,
    replaced by what compares greater."""
    dtype, npdt = (cad.F16, np.float16) if dtype_name == "f16" else (cad.F32, np.float32)
    ops = [Op("maxpool", "pool", 0, 1, k=k, stride=1, pad=pad), Op("concat", "cat", 0, 2, srcs=(0, 0)),
           Op("conv", "a", 1, 3, 8, 8, 1, 1, 0, 0.5, False), Op("conv", "b", 2, 4, 16, 8, 1, 1, 0, 0.5, False)]
    n, h, w = 2, 9, 11
    x, ws, bs = wl.net_tensors(ops, "nan-pool", (n, 8, h, w))
    rng = np.random.default_rng(k * 7 + pad)
    x[rng.random(x.shape) < 0.25] = np.nan
    x[rng.random(x.shape) < 0.1] = np.inf
    x[rng.random(x.shape) < 0.1] = -np.inf
    x[0, 0], x[1, 3, :6, :6] = np.nan, np.nan
    x = x.astype(npdt)
    ho, wo = h + 2 * pad - k + 1, w + 2 * pad - k + 1
    want = np.zeros((n, 8, ho, wo), npdt)
    for r in range(ho):
        for c in range(wo):
            m = None
            for a in range(max(r - pad, 0), min(r - pad + k, h)):
                for b in range(max(c - pad, 0), min(c - pad + k, w)):
                    m = x[:, :, a, b] if m is None else np.where(x[:, :, a, b] > m, x[:, :, a, b], m)
            want[:, :, r, c] = m
    for pin in (None, "cl_mfma_64x64_s3"):
        net = cad.build_net(ops, ws, bs, (n, 8, h, w), dtype, use_graph=False)
        if pin:
            net.set_op_variant(2, pin)
        net.run(torch.from_numpy(x).cuda())
        torch.cuda.synchronize()
        assert np.array_equal(net.read_buffer(1, want.shape), want, equal_nan=True), pin
        assert np.array_equal(net.read_buffer(2, (n, 16, h, w)), np.concatenate([x, x], 1), equal_nan=True), pin
        net.free()


@pytest.mark.parametrize("hw", [(7, 7), (1, 1), (5, 9), (8, 8), (13, 11), (33, 40)])
def test_global_pool_sums_are_as_exact_as_on_planes(cad, hw):
    """The mean of a map of positive values, against 64 bits and against the pool on planes over the same map."""
    ops = [Op("conv", "a", 0, 1, 32, 512, 1, 1, 0, 0.5, True), Op("avgpool", "gap", 1, 2)]
    shape = (4, 32) + hw
    x, ws, bs = wl.net_tensors(ops, "gap-sums", shape, input_relu=True)
    net = cad.build_net(ops, ws, bs, shape, cad.F32, use_graph=False)
    net.set_op_variant(0, "cl_mfma_64x64_s3")
    y = net.run(torch.from_numpy(x).cuda()).cpu().numpy().reshape(4, 512).astype(np.float64)
    torch.cuda.synchronize()
    mid = net.read_buffer(1, (4, 512) + hw)
    net.free()
    planes = cad.cadnn_global_avgpool(torch.from_numpy(mid).cuda()).cpu().numpy().reshape(4, 512).astype(np.float64)
    ref = mid.astype(np.float64).mean((2, 3))
    off = lambda g: float(np.sqrt(((g - ref) ** 2).sum() / (ref ** 2).sum()))
    assert off(y) <= 1.1 * off(planes) + 1e-9, (off(y), off(planes))
    # any chain of hw / 64 + 1 additions, 7 levels and the division
    assert (np.abs(y - ref) <= (hw[0] * hw[1] // 64 + 9) * 2.0 ** -24 * np.abs(mid).astype(np.float64).mean((2, 3))).all()


def test_split_tiles_pinned_and_run_at_once_on_another_stream(cad):
    """The arrival counters of a split K are zero for a launch on a non-blocking stream right behind the pin, with the
    scratch growing and the tiles changing in between."""
    ops = [Op("conv", "a", 0, 1, 64, 64, 3, 1, 1, 0.5, True), Op("conv", "b", 1, 2, 64, 64, 3, 1, 1, 0.5, False)]
    shape = (2, 64, 30, 31)
    x, ws, bs = wl.net_tensors(ops, "split-stream", shape, input_relu=True)
    ref, ins, outs = oracle.run_net(ops, x, ws, bs, dtype=np.float32)
    bound = chain_bounds(ops, ins, outs, ws, bs, False)[-1]
    xd = torch.from_numpy(x).cuda()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    for names in (("cl_mfma_64x64_s3k2", "cl_mfma_64x64_s3k4"), ("cl_mfma_64x64_s4k4", "cl_mfma_64x64_s3k2"), ("cl_mfma_64x64_s3", "cl_mfma_64x64_s3k4")):
        net = cad.build_net(ops, ws, bs, shape, cad.F32, use_graph=False)
        with torch.cuda.stream(stream):
            for i, name in enumerate(names):
                net.set_op_variant(i, name)
            got = [net.run(xd) for _ in range(3)]
        stream.synchronize()
        for y in got:
            assert_within_bound(y.cpu().numpy(), ref, bound, str(names))
        net.free()


def test_a_refused_name_changes_nothing(cad):
    """A name that no variant of the op has, or one of the other execution that does not serve the op, is refused
    and leaves the net in the execution, and with the choices, it had."""
    ops, shape = deep_net()
    x, ws, bs = wl.net_tensors(ops, "refused", shape, input_relu=True)
    xd = torch.from_numpy(x).cuda()
    net = cad.build_net(ops, ws, bs, shape, cad.F32, use_graph=True)
    planes = net.variants()
    assert not planes[0].startswith("cl_")
    want = net.run(xd)
    for op, name in ((0, "no_such_kernel"), (0, "cl_no_such_tile"), (4, "cl_mfma_64x64")):
        with pytest.raises(cad.CadnnError):
            net.set_op_variant(op, name)
        assert net.variants() == planes
    small = [Op("conv", "a", 0, 1, 16, 16, 1, 1, 0, 0.5, True), Op("conv", "b", 1, 2, 16, 16, 3, 1, 1, 0.5, True)]
    _, sw, sb = wl.net_tensors(small, "refused-small", (1, 16, 9, 9))
    # (16 channels are too few for the large tile, one K step too few for two slices)
    little = cad.build_net(small, sw, sb, (1, 16, 9, 9), cad.F32, use_graph=False)
    before = little.variants()
    for name in ("cl_mfma_128x128_s2", "cl_mfma_64x64_s3k2"):
        with pytest.raises(cad.CadnnError):
            little.set_op_variant(0, name)
        assert little.variants() == before
    little.free()
    assert torch.equal(net.run(xd), want)
    net.set_op_variant(1, "cl_mfma_64x64_s4k4")
    tiles = net.variants()
    want = net.run(xd)
    # (a name of the plane layouts that the 3x3 layer has no use for: a kernel of 1x1 filters)
    probe = cad.build_net(ops, ws, bs, shape, cad.F32, use_graph=False)
    foreign = sorted(set(probe.op_candidates(0)) - set(probe.op_candidates(1)))
    probe.free()
    assert foreign
    for name in ("no_such_kernel", foreign[0], "apart", "cl_mfma_64x64"):
        with pytest.raises(cad.CadnnError):
            net.set_op_variant(1, name)
        assert net.variants() == tiles, name
    assert torch.equal(net.run(xd), want)
    torch.cuda.synchronize()
    net.free()


def test_finalize_again_after_a_pin(cad):
    """A net that a pin took channels-last is finalized a second time with a workspace of exactly the size asked
    for (smaller than the channels-last tensors, whose few channels are padded): nothing behind it is written,
    the first workspace is not used any more, the pin stays, and a plane variant takes the net to the new one."""
    import ctypes
    ops = [Op("conv", "stem", 0, 1, 3, 8, 3, 1, 1, 0.0, True), Op("conv", "a", 1, 2, 8, 8, 3, 1, 1, 0.5, True),
           Op("conv", "b", 2, 3, 8, 4, 1, 1, 0, 0.5, False), Op("avgpool", "gap", 3, 4)]
    shape = (2, 3, 40, 37)
    x, ws, bs = wl.net_tensors(ops, "again", shape)
    ref, ins, outs = oracle.run_net(ops, x, ws, bs, dtype=np.float32)
    bound = chain_bounds(ops, ins, outs, ws, bs, False)[-1]
    xd = torch.from_numpy(x).cuda()
    net = cad.build_net(ops, ws, bs, shape, cad.F32, use_graph=False)
    planes = net.variants()
    net.set_op_variant(0, "cl_mfma_64x64_s3")
    first = net._keep[-1]
    size = first.numel()
    assert not planes[0].startswith("cl_")

    def check(what):
        y = net.run(xd)
        torch.cuda.synchronize()
        assert_within_bound(y.cpu().numpy(), ref, bound, what)

    check("pinned")
    for again in range(2):
        room = torch.full((size + (4 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        cad.binding._check(cad.lib().cadnn_net_finalize(net.handle, ctypes.c_void_p(room.data_ptr()), size, 0))
        first.fill_(0x7F)                       # (what the caller does with a workspace it has taken back)
        first = room
        check("finalized again")
        assert net.op_variant(0) == "cl_mfma_64x64_s3"
        assert bool((room[size:] == 0x5A).all())
    net.set_variants(planes)
    check("back on planes")
    assert net.variants() == planes and bool((first[size:] == 0x5A).all())
    net.set_op_variant(0, "cl_mfma_64x64_s4")
    check("channels-last once more")
    # other flags lay the net out anew: no pin is left
    room = torch.empty(size, dtype=torch.uint8, device="cuda")
    cad.binding._check(cad.lib().cadnn_net_finalize(net.handle, ctypes.c_void_p(room.data_ptr()), size, 4))
    check("plain layout")
    assert not net.op_variant(0).startswith("cl_")
    net.free()
