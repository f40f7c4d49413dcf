"""A layer's passes in one call each (xconv_layer_fwd, xconv_layer_bwd) give the results of the separate calls bit for bit: the same
kernels run, with the packing of the weights and the sum of the bias gradient's pieces carried by other launches.  Bias gradients of
one piece and of several, input gradients of one class, of four and of more than one launch takes, weights of several tiles."""
import ctypes

import pytest
import torch

from paper_2106_06998_amd import binding as xb
from test_gpu_conv import DEV, TD, say

pytestmark = pytest.mark.gpu

# B, C_in, C_out, H, W, k, stride, pad, r, channels-last; all but the first sum their bias gradient from several pieces (each at
# least 32 KB of a channel's values, or of all of them in channels-last)
CASES = [
    (2, 16, 24, 12, 12, 3, 1, 1, 8, False),
    (8, 24, 20, 64, 64, 3, 1, 1, 8, False),
    (9, 40, 72, 128, 130, 3, 2, 1, 16, False),
    (32, 32, 9, 100, 98, 3, 3, 0, 8, False),       # nine classes
    (4, 48, 36, 60, 61, 5, 4, 2, 16, True),        # sixteen
    (8, 136, 150, 40, 40, 3, 1, 1, 32, True),      # chunks of channels
    (6, 64, 40, 50, 52, 1, 1, 0, 16, True),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("mode", [0, 1], ids=["channel", "multi"])
@pytest.mark.parametrize("case", CASES, ids=["c%d-%d-%dx%d-k%d-s%d" % c[1:7] for c in CASES])
def test_passes_are_those_of_the_separate_calls(case, mode, dtype):
    B, C_in, C_out, H, W, k, s, p, r, cl = case
    say("layer passes %s %s mode %d" % (case, dtype, mode))
    Ho, Wo = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1
    assert case is CASES[0] or B * Ho * Wo * 2 * (C_out if cl else 1) >= 65536
    L, td = xb.lib(), TD[dtype]
    fmt = torch.channels_last if cl else torch.contiguous_format
    g = torch.Generator(device=DEV).manual_seed(31)

    def normal(*shape):
        t = torch.randn(shape, device=DEV, generator=g).to(td)
        return t.contiguous(memory_format=fmt) if len(shape) == 4 and shape[1:] != (C_in, k, k) else t

    x, w, bias, dy = normal(B, C_in, H, W), normal(C_out, C_in, k, k), normal(C_out), normal(B, C_out, Ho, Wo)
    d = xb.make_desc(B, C_in, C_out, H, W, k, s, p, r, dtype, "rademacher", 17, xb.XCONV_NHWC if cl else xb.XCONV_NCHW)
    P = ctypes.byref(d)

    def filled(*shape):
        t = torch.full(shape, float("nan"), dtype=td, device=DEV)
        return t.contiguous(memory_format=fmt) if shape[1:] != (C_in, k, k) and len(shape) == 4 else t

    def scratch(n):
        return torch.full((max(int(n), 16),), 0xff, dtype=torch.uint8, device=DEV)

    L.xconv_layer_workspace_bytes.restype = ctypes.c_size_t
    for f in (L.xconv_layer_fwd, L.xconv_layer_bwd):
        f.restype = ctypes.c_int
    vp, sz = ctypes.c_void_p, ctypes.c_size_t
    state_bytes = int(xb.xconv_xt_bytes(d) if mode == 0 else xb.xconv_pixel_xbar_bytes(d))
    states, outs = [], []
    for one in (True, False):
        state = scratch(state_bytes)
        y, dx, dw, db = filled(B, C_out, Ho, Wo), filled(B, C_in, H, W), filled(C_out, C_in, k, k), filled(C_out)
        if one:
            ws = scratch(L.xconv_layer_workspace_bytes(P, mode, 0))
            assert L.xconv_layer_fwd(P, mode, vp(x.data_ptr()), vp(w.data_ptr()), vp(bias.data_ptr()), vp(y.data_ptr()), vp(state.data_ptr()), vp(ws.data_ptr()), sz(ws.numel()), vp(0)) == 0
            wb = scratch(L.xconv_layer_workspace_bytes(P, mode, 1))
            assert L.xconv_layer_bwd(P, mode, vp(dy.data_ptr()), vp(w.data_ptr()), vp(state.data_ptr()), vp(dx.data_ptr()), vp(dw.data_ptr()), xb.DTYPES[dtype], vp(db.data_ptr()),
                                     vp(wb.data_ptr()), sz(wb.numel()), vp(0)) == 0
        else:
            xb.xconv_conv_fwd_ws(d, x, w, bias, y, scratch(xb.xconv_conv_workspace_bytes(d, 0)))
            xb.xconv_dx_exact_ws(d, dy, w, dx, scratch(xb.xconv_conv_workspace_bytes(d, 1)))
            xb.xconv_bias_grad(d, dy, db, scratch(xb.xconv_bias_workspace_bytes(d)))
            if mode == 0:
                xb.xconv_probe_fwd(d, x, state, None, scratch(xb.xconv_workspace_bytes(d, xb.XCONV_OP_PROBE)))
                xb.xconv_dw_estimate_as(d, dy, state, None, dw, xb.DTYPES[dtype], scratch(xb.xconv_workspace_bytes(d, xb.XCONV_OP_ESTIMATE)))
            else:
                xb.xconv_pixel_probe_fwd(d, x, state, scratch(xb.xconv_pixel_workspace_bytes(d, xb.XCONV_OP_PROBE)))
                xb.xconv_pixel_dw_estimate_as(d, dy, state, dw, xb.DTYPES[dtype], scratch(xb.xconv_pixel_workspace_bytes(d, xb.XCONV_OP_ESTIMATE)))
        torch.cuda.synchronize()
        states.append(state)
        outs.append((y, dx, dw, db))
    assert torch.equal(states[0], states[1])
    for name, a, b in zip(("y", "dX", "dW", "db"), *outs):
        assert not bool(torch.isnan(a).any()), name
        assert torch.equal(a, b), name
    # and the separate bias gradient is the sum (fp32 sums, one rounding)
    want = dy.double().sum((0, 2, 3))
    tol = {"f32": 0.0, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype] * want.abs() + 1e-5 * dy.double().abs().sum((0, 2, 3))
    assert bool(((outs[0][3].double() - want).abs() <= tol).all())
