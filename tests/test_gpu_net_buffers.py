"""A captured net serves whatever input and output tensors a call brings: the launches that touch them
stay outside the replayed graph."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype_name", ["f32", "f16"])
@pytest.mark.parametrize("blocks,cl", [(1, False), (3, False), (3, True)])
def test_new_tensors_on_every_call(blocks, cl, dtype_name):
    """blocks = 1: every launch touches the caller's tensors or stands alone (no graph); 3: the input is
    read by a residual in the middle, the graph is the longest run behind it.  Bit-equal to the net
    without a graph, with eager work and allocations in between."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1905_00571_amd as cad
    dtype, npdt = (cad.F16, np.float16) if dtype_name == "f16" else (cad.F32, np.float32)
    ops = []
    for b in range(blocks):
        src = 3 * b
        ops += [wl.Op("conv", f"a{b}", src, src + 1, 64, 16, 1, 1, 0, 0.8, True),
                wl.Op("conv", f"b{b}", src + 1, src + 2, 16, 16, 3, 1, 1, 0.8, True),
                wl.Op("conv", f"c{b}", src + 2, src + 3, 16, 64, 1, 1, 0, 0.8, True, res=src)]
    shape = (2, 64, 13, 14)
    x, ws, bs = wl.net_tensors(ops, "buffers", shape, input_relu=True)
    net = cad.build_net(ops, ws, bs, shape, dtype, use_graph=True)
    eager = cad.build_net(ops, ws, bs, shape, dtype, use_graph=False)
    if cl:
        for n in (net, eager):
            n.set_op_variant(0, "cl_mfma_64x64_s3")
    kept = []
    for rep in range(5):
        xi = torch.from_numpy(np.roll(x, rep, axis=2).astype(npdt)).cuda()
        want = eager.run(xi)
        got = net.run(xi)
        kept.append((xi, got, want))              # the buffers stay in use: every call gets new ones
        torch.randn(1000, device="cuda").sum()
    for rep, (xi, got, want) in enumerate(kept):
        assert torch.equal(got, want), rep
    again = net.run(kept[1][0], kept[3][1])       # and old ones in another combination
    torch.cuda.synchronize()
    assert torch.equal(again, kept[1][2])
    net.free()
    eager.free()
