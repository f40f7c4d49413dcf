"""The library enqueues on the stream it is given and allocates nothing, so a layer runs the same on
a side stream and inside a captured HIP graph: both against the eager result on the default stream,
which the parity tests check against the oracle (results are deterministic, hence bit-equal)."""
import numpy as np
import pytest
import torch

from paper_2106_06998_amd import binding as xb
from paper_2106_06998_amd import synth
from test_gpu_parity import DEV, say

pytestmark = pytest.mark.gpu

LAYERS = [
    ("f32", 6, 32, 48, 17, 15, 3, 1, 1, 16, "gaussian"),       # fp32 producer/consumer kernel
    ("f16", 9, 64, 64, 14, 14, 3, 1, 1, 64, "rademacher"),     # 16-bit producer/consumer kernel
    ("bf16", 3, 20, 18, 7, 9, 3, 2, 1, 20, "rademacher"),      # ragged planes: probe on the matrix cores, repacked dY
    ("bf16", 3, 20, 18, 7, 9, 3, 1, 1, 20, "gaussian"),        # ... in fp32 arithmetic, Z in fragment order from a launch in front
    ("f16", 3, 528, 18, 7, 9, 3, 2, 1, 20, "rademacher"),      # generic probe, Z through the workspace between two launches
]


class Layer:
    def __init__(self, e):
        dtype, B, C_in, C_out, H, W, k, st, pad, r, probe = e
        self.e = e
        self.d = xb.make_desc(B, C_in, C_out, H, W, k, st, pad, r, dtype, probe, 99)
        Ho, Wo = (H + 2 * pad - k) // st + 1, (W + 2 * pad - k) // st + 1
        self.X = xb.to_device(synth.draw((B, C_in, H, W), 31, "relu_normal", 1.0, dtype), dtype, DEV)
        self.dY = xb.to_device(synth.draw((B, C_out, Ho, Wo), 32, "normal", 1e-2, dtype), dtype, DEV)
        self.Xt = xb.alloc_xt(self.d, DEV)
        self.dW = torch.empty((C_out, C_in, k, k), dtype=torch.float32, device=DEV)
        self.wsp = xb.alloc_ws(self.d, xb.XCONV_OP_PROBE, DEV)
        self.wse = xb.alloc_ws(self.d, xb.XCONV_OP_ESTIMATE, DEV)

    def step(self, stream=None):
        xb.xconv_probe_fwd(self.d, self.X, self.Xt, None, self.wsp, stream)
        xb.xconv_dw_estimate(self.d, self.dY, self.Xt, None, self.dW, self.wse, stream)

    def refill(self, salt):
        dtype, B, C_in, C_out, H, W, k, st, pad, r, probe = self.e
        self.X.copy_(xb.to_device(synth.draw(tuple(self.X.shape), 41 + salt, "relu_normal", 1.0, dtype), dtype, DEV))
        self.dY.copy_(xb.to_device(synth.draw(tuple(self.dY.shape), 51 + salt, "normal", 1e-2, dtype), dtype, DEV))


@pytest.mark.parametrize("e", LAYERS, ids=["%s-%d-%s" % (e[0], e[1], e[10]) for e in LAYERS])
def test_side_stream_gives_the_default_stream_result(e):
    say("side stream %s" % (e,))
    L = Layer(e)
    L.step()
    torch.cuda.synchronize()
    want = L.dW.clone()
    L.dW.fill_(float("nan"))
    L.Xt.fill_(0x7f)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    L.step(side)                        # explicit stream argument, not the current stream
    side.synchronize()
    assert torch.equal(L.dW, want)
    L.dW.fill_(float("nan"))
    torch.cuda.synchronize()
    with torch.cuda.stream(side):       # the binding's default: torch's current stream
        L.step()
    side.synchronize()
    assert torch.equal(L.dW, want)


@pytest.mark.parametrize("e", LAYERS, ids=["%s-%d-%s" % (e[0], e[1], e[10]) for e in LAYERS])
def test_captured_graph_replays_give_the_eager_result(e):
    say("graph capture %s" % (e,))
    L = Layer(e)
    L.step()                            # eager once: kernel attributes are set outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        L.step()
    for salt in range(3):               # new inputs in the same buffers, eager work and synchronisation between replays
        L.refill(salt)
        L.step()
        torch.cuda.synchronize()
        want = L.dW.clone()
        L.dW.fill_(float("nan"))
        L.Xt.fill_(0x7f)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(L.dW, want), salt
        assert bool(torch.isfinite(L.dW).all())


def test_layers_reach_the_kernels_they_stand_for():
    names = []
    for e in LAYERS:
        L = Layer(e)
        xb.xconv_prof_enable(True)
        xb.xconv_prof_collect()
        L.step()
        torch.cuda.synchronize()
        names.append({xb.xconv_prof_kernel_name(k) for k, _ in xb.xconv_prof_collect()})
        xb.xconv_prof_enable(False)
    assert "probe_generic_kernel" not in set().union(*names[:4])
    assert {"probe_generic_kernel", "gen_z_kernel", "repack_planes_kernel"} <= names[4], names[4]
    assert {"pack_z_kernel"} <= names[3] and "repack_planes_kernel" in names[2], names


def test_two_layers_on_two_streams_at_once():
    # the library keeps no state between calls: layers with buffers of their own, enqueued alternately on two
    # streams, give what each gives alone
    say("two streams at once")
    a, b = Layer(LAYERS[0]), Layer(LAYERS[1])
    a.step()
    b.step()
    torch.cuda.synchronize()
    want_a, want_b = a.dW.clone(), b.dW.clone()
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    for rep in range(4):
        a.dW.fill_(float("nan"))
        b.dW.fill_(float("nan"))
        torch.cuda.synchronize()
        xb.xconv_probe_fwd(a.d, a.X, a.Xt, None, a.wsp, sa)
        xb.xconv_probe_fwd(b.d, b.X, b.Xt, None, b.wsp, sb)
        xb.xconv_dw_estimate(a.d, a.dY, a.Xt, None, a.dW, a.wse, sa)
        xb.xconv_dw_estimate(b.d, b.dY, b.Xt, None, b.dW, b.wse, sb)
        sa.synchronize()
        sb.synchronize()
        assert torch.equal(a.dW, want_a) and torch.equal(b.dW, want_b), rep



@pytest.mark.parametrize("packed", [True, False], ids=["packed", "gathered"])
@pytest.mark.parametrize("e", [("f32", 4, 16, 24, 30, 3, 1, 1), ("f16", 3, 20, 40, 33, 3, 5, 1), ("bf16", 2, 24, 9, 28, 4, 4, 0)],
                         ids=["s1", "cleared", "sixteen-classes"])
def test_captured_products_replay_the_eager_result(e, packed):
    # forward product and input gradient, among them strided ones whose dX is cleared by a kernel in front
    dtype, B, C_in, C_out, n, k, s, p = e
    say("graph capture of the products %s packed %s" % (e, packed))
    td, m = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype], (n + 2 * p - k) // s + 1
    d = xb.make_desc(B, C_in, C_out, n, n, k, s, p, 1, dtype)
    g = torch.Generator(device=DEV).manual_seed(5)
    x, w, dy = (torch.empty(shape, dtype=td, device=DEV) for shape in ((B, C_in, n, n), (C_out, C_in, k, k), (B, C_out, m, m)))
    y, dx = torch.empty_like(dy), torch.empty_like(x)
    ws = [xb.alloc_bytes(xb.xconv_conv_workspace_bytes(d, t)) if packed else None for t in (0, 1)]

    def step():
        xb.xconv_conv_fwd_ws(d, x, w, None, y, ws[0])
        xb.xconv_dx_exact_ws(d, dy, w, dx, ws[1])

    def refill():
        for t in (x, w, dy):
            t.normal_(generator=g)

    refill()
    step()                              # eager once: kernel attributes are set outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(3):
        refill()
        step()
        torch.cuda.synchronize()
        want = y.clone(), dx.clone()
        y.fill_(float("nan"))
        dx.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want[0]) and torch.equal(dx, want[1]), rep
        assert bool(torch.isfinite(dx).all())
