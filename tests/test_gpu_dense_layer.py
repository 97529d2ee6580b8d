"""cadnn_dense_conv2d over the sizes where its two routes and their tiles end: channels and pixels
around the 64 and 128 of a tile and the 64 bytes of a step, halos, strides, rectangular filters, K
long enough to be split, too few channels for the channels-last route.  The bound holds for any
order of fp32 sums of K products: (K + 3) 2^-24 (sum |w| |x| + |b| + |r|), plus one rounding to storage."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

#        n  cin cout  h   w  kh kw stride pad residual
CASES = [(1, 16, 1, 1, 1, 1, 1, 1, 0, False),
         (2, 17, 65, 9, 5, 3, 3, 1, 1, True),
         (3, 33, 130, 7, 7, 1, 1, 1, 0, True),
         (1, 64, 64, 8, 8, 3, 3, 1, 1, False),
         (1, 512, 64, 7, 7, 3, 3, 1, 1, True),      # K split over workgroups
         (2, 100, 24, 13, 11, 5, 5, 1, 2, False),
         (1, 40, 40, 17, 17, 7, 7, 2, 3, True),
         (4, 48, 129, 31, 33, 1, 7, 1, 3, False),
         (2, 96, 72, 14, 10, 3, 3, 2, 0, False),
         (32, 64, 128, 14, 14, 3, 3, 1, 1, True),   # the large tiles
         (2, 3, 24, 21, 21, 7, 7, 2, 3, False),     # the kernel on planes
         (1, 15, 8, 6, 6, 9, 9, 1, 4, True)]


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("case", CASES)
def test_dense_layer_against_64_bits(case, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1905_00571_amd as cad
    n, cin, cout, h, w, kh, kw, stride, pad, residual = case
    tt = torch.float16 if dtype == "f16" else torch.float32
    gen = torch.Generator().manual_seed(cin * 131 + cout)
    x = torch.randn(n, cin, h, w, generator=gen).to(tt)
    wt = (torch.randn(cout, cin, kh, kw, generator=gen) * (2.0 / (cin * kh * kw)) ** 0.5).to(tt)
    b = torch.randn(cout, generator=gen)
    conv = torch.nn.functional.conv2d
    ref = conv(x.double(), wt.double(), b.double(), stride, pad)
    size = conv(x.double().abs(), wt.double().abs(), b.double().abs(), stride, pad)
    r = None
    if residual:
        r = torch.randn(ref.shape, generator=gen).to(tt)
        ref, size = ref + r.double(), size + r.double().abs()
    ref = ref.clamp_min(0.0)
    got = cad.cadnn_dense_conv2d(wt.cuda(), x.cuda(), stride, pad, b.cuda(), None if r is None else r.cuda(), True)
    got = got.cpu().double()
    bound = (cin * kh * kw + 3) * 2.0 ** -24 * size
    if dtype == "f16":
        bound = bound + 2.0 ** -11 * ref.abs() + 2.0 ** -25
    excess = ((got - ref).abs() - bound).max().item()
    assert got.shape == ref.shape and excess <= 0.0, f"{case} {dtype}: {excess:.3e} above the bound"


@pytest.mark.parametrize("cin,cout,h,w,k,stride", [(33, 40, 9, 11, 3, 1), (64, 130, 12, 10, 3, 2), (512, 70, 7, 7, 3, 1), (160, 1, 15, 13, 5, 1)])
def test_dense_layer_of_non_finite_values_in_a_used_workspace(cin, cout, h, w, k, stride):
    """fp32: infinities and NaN come out where 64-bit arithmetic has them and nowhere else, in a workspace where the call
    before left NaN (the rows behind the last filter are not written, and must not count)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1905_00571_amd as cad
    gen = torch.Generator().manual_seed(cin + cout)
    x = torch.randn(2, cin, h, w, generator=gen)
    wt = torch.randn(cout, cin, k, k, generator=gen) * (2.0 / (cin * k * k)) ** 0.5
    b = torch.randn(cout, generator=gen)
    wide = (cout + 127) // 128 * 128
    conv = torch.nn.functional.conv2d
    for bad in (False, True):
        if bad:
            x[0, 1, 0, 0], x[0, cin - 1, h - 1, w - 1], x[1, 0, h // 2, w // 2] = float("inf"), float("-inf"), float("nan")
        cad.cadnn_release_workspaces()
        cad.cadnn_dense_conv2d(torch.full((wide, cin, k, k), float("nan")).cuda(), torch.full_like(x, float("nan")).cuda(), stride, k // 2)
        got = cad.cadnn_dense_conv2d(wt.cuda(), x.cuda(), stride, k // 2, b.cuda()).cpu()
        ref = conv(x.double(), wt.double(), b.double(), stride, k // 2)
        size = conv(x.double().abs(), wt.double().abs(), b.double().abs(), stride, k // 2)
        finite = torch.isfinite(ref)
        assert bool(finite.all()) != bad
        assert torch.equal(torch.nan_to_num(got[~finite], 1.0, 2.0, 3.0), torch.nan_to_num(ref[~finite].float(), 1.0, 2.0, 3.0))
        excess = ((got.double() - ref).abs() - (cin * k * k + 3) * 2.0 ** -24 * size)[finite].max().item()
        assert excess <= 0.0, f"{excess:.3e} above the bound"


def test_dense_layer_repeats_and_follows_new_weights():
    """Nothing of a call is kept for the next: new weights and inputs in the same tensors."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1905_00571_amd as cad
    x, wt = torch.randn(2, 64, 14, 14).cuda(), torch.randn(64, 64, 3, 3).cuda()
    first = cad.cadnn_dense_conv2d(wt, x, 1, 1).clone()
    assert torch.equal(first, cad.cadnn_dense_conv2d(wt, x, 1, 1))
    wt.mul_(2.0)
    assert torch.equal(2.0 * first, cad.cadnn_dense_conv2d(wt, x, 1, 1))
    x.mul_(0.5)
    assert torch.equal(first, cad.cadnn_dense_conv2d(wt, x, 1, 1))


def test_dense_layer_workspaces_on_two_streams_threads_and_under_capture():
    """Workspaces are handed from call to call: calls that alternate between streams and threads, with
    growing and shrinking sizes, and a captured graph's replays give what calls one by one give."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import threading
    import paper_1905_00571_amd as cad
    gen = torch.Generator().manual_seed(3)
    layers = []
    for cin, cout, hw, k in ((64, 64, 28, 3), (256, 128, 14, 3), (32, 48, 56, 5), (512, 64, 7, 3)):
        x = torch.randn(4, cin, hw, hw, generator=gen).half().cuda()
        w = (torch.randn(cout, cin, k, k, generator=gen) * 0.05).half().cuda()
        layers.append((w, x, k // 2))
    want = []
    for w, x, pad in layers:
        want.append(cad.cadnn_dense_conv2d(w, x, 1, pad).clone())
        torch.cuda.synchronize()
    failures = []

    def work(seed):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for i in range(40):
                j = (i * (seed + 1) + seed) % len(layers)
                w, x, pad = layers[j]
                y = cad.cadnn_dense_conv2d(w, x, 1, pad)
                if not torch.equal(y, want[j]):
                    failures.append((seed, i, j))
        stream.synchronize()

    threads = [threading.Thread(target=work, args=(s,)) for s in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failures
    # a captured graph keeps to the kernels on planes (another order of the same fp32 sums)
    w, x, pad = layers[0][0].float(), layers[0][1].float(), layers[0][2]
    eager = cad.cadnn_dense_conv2d(w, x, 1, pad).clone()
    y = torch.empty_like(eager)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cad.cadnn_dense_conv2d(w, x, 1, pad, out=y)
    bound = 2 * (w[0].numel() + 3) * 2.0 ** -24 * torch.nn.functional.conv2d(x.double().abs().cpu(), w.double().abs().cpu(), None, 1, pad)
    for _ in range(3):
        y.zero_()
        graph.replay()
        cad.cadnn_dense_conv2d(layers[1][0], layers[1][1], 1, layers[1][2])
        torch.cuda.synchronize()
        assert bool(((y.double() - eager.double()).abs().cpu() <= bound).all())


def test_kept_workspaces_are_given_back():
    """Some 30 MiB a call stay for later calls; cadnn_release_workspaces returns them, also right behind a call
    whose kernels still run, and the next call takes a new one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1905_00571_amd as cad
    x, wt = torch.randn(4, 128, 110, 110).cuda(), torch.randn(64, 128, 3, 3).cuda()
    want = cad.cadnn_dense_conv2d(wt, x, 1, 1)
    y = torch.empty_like(want)
    torch.cuda.synchronize()
    cad.cadnn_release_workspaces()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for _ in range(3):
        y.zero_()
        cad.cadnn_dense_conv2d(wt, x, 1, 1, out=y)
        cad.cadnn_release_workspaces()
        torch.cuda.synchronize()
        assert torch.equal(y, want)
    cad.cadnn_dense_conv2d(wt, x, 1, 1, out=y)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] <= free - (24 << 20)
    cad.cadnn_release_workspaces()
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] >= free - (4 << 20)


def test_workspaces_of_large_fp32_weights_are_kept():
    """56 MiB of weights take 84 at the 6 bytes of their device form: held for the next call like 64 MiB of others."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1905_00571_amd as cad
    x, wt = torch.randn(1, 1600, 7, 7).cuda(), (torch.randn(1024, 1600, 3, 3) * 0.01).cuda()
    y = cad.cadnn_dense_conv2d(wt, x, 1, 1)
    torch.cuda.synchronize()
    cad.cadnn_release_workspaces()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    cad.cadnn_dense_conv2d(wt, x, 1, 1, out=y)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] <= free - (80 << 20)
    cad.cadnn_release_workspaces()
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] >= free - (4 << 20)


class _PoolLocation(ctypes.Structure):
    _fields_ = [("type", ctypes.c_int), ("id", ctypes.c_int)]


class _PoolProps(ctypes.Structure):
    _fields_ = [("alloc_type", ctypes.c_int), ("handle_types", ctypes.c_int), ("location", _PoolLocation),
                ("security", ctypes.c_void_p), ("max_size", ctypes.c_size_t), ("reserved", ctypes.c_ubyte * 56)]


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_without_memory_for_a_workspace(dtype):
    """A device memory pool that may hold 2 MiB: a layer whose workspace needs more runs on the tensors as they
    are, and the next one, with memory, on its workspace again."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1905_00571_amd as cad
    tt = torch.float16 if dtype == "f16" else torch.float32
    gen = torch.Generator().manual_seed(5)
    x = torch.randn(2, 72, 60, 61, generator=gen).to(tt).cuda()
    wt = (torch.randn(40, 72, 3, 3, generator=gen) * 0.05).to(tt).cuda()
    with_room = cad.cadnn_dense_conv2d(wt, x, 1, 1).clone()
    torch.cuda.synchronize()
    cad.cadnn_release_workspaces()
    hip = ctypes.CDLL("libamdhip64.so")
    hip.hipDeviceSetMemPool.argtypes = [ctypes.c_int, ctypes.c_void_p]
    hip.hipMemPoolDestroy.argtypes = [ctypes.c_void_p]
    before, small = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipDeviceGetMemPool(ctypes.byref(before), 0) == 0
    props = _PoolProps(alloc_type=1, handle_types=0, location=_PoolLocation(1, 0), security=None, max_size=2 << 20)
    assert hip.hipMemPoolCreate(ctypes.byref(small), ctypes.byref(props)) == 0
    assert hip.hipDeviceSetMemPool(0, small) == 0
    try:
        p = ctypes.c_void_p()
        refused = hip.hipMallocAsync(ctypes.byref(p), ctypes.c_size_t(8 << 20), None) != 0
        hip.hipGetLastError()
        got = [cad.cadnn_dense_conv2d(wt, x, 1, 1).clone() for _ in range(2)]
        torch.cuda.synchronize()
        if not refused:
            hip.hipFree(p)
        cad.cadnn_release_workspaces()
    finally:
        assert hip.hipDeviceSetMemPool(0, before) == 0
        hip.hipMemPoolDestroy(small)
    assert refused, "the pool's limit is not enforced here: nothing was tested"
    conv = torch.nn.functional.conv2d
    size = conv(x.double().abs().cpu(), wt.double().abs().cpu(), None, 1, 1)
    ref = conv(x.double().cpu(), wt.double().cpu(), None, 1, 1)
    bound = (72 * 9 + 3) * 2.0 ** -24 * size
    if dtype == "f16":
        bound = bound + 2.0 ** -11 * ref.abs() + 2.0 ** -25
    for y in got + [with_room]:
        assert bool(((y.double().cpu() - ref).abs() <= bound).all())
    assert torch.equal(cad.cadnn_dense_conv2d(wt, x, 1, 1), with_room)
