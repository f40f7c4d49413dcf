"""The bias gradient (xconv_bias_grad) against fp64 sums of the same storage values: one piece and several, planes that are whole
16-byte vectors and planes that are not, planes smaller than a workgroup's stride, both layouts, a misaligned tensor; and the
weight gradient stored in a 16-bit type (xconv_dw_estimate_as, xconv_pixel_dw_estimate_as), which is the fp32 one rounded once."""
import numpy as np
import pytest
import torch

from paper_2106_06998_amd import binding as xb
from paper_2106_06998_amd import synth
from test_gpu_conv import DEV, TD, say

pytestmark = pytest.mark.gpu

# B, C, H, W, dtype, channels-last, elements the tensor starts past a 16-byte boundary
CASES = [
    (3, 5, 7, 9, "f32", False, 0),
    (4, 600, 8, 8, "f16", False, 0),         # one piece per channel
    (2, 3, 64, 64, "bf16", False, 0),        # several pieces per channel
    (300, 2, 1, 1, "f32", False, 0),         # planes of one value
    (2, 4, 33, 31, "f16", False, 1),
    (5, 24, 9, 10, "bf16", True, 0),
    (3, 7, 11, 5, "f16", True, 0),           # channels that are no whole vectors
    (1, 2052, 3, 3, "f32", True, 0),         # more channels than one workgroup spans
    (2, 40, 40, 40, "f32", True, 0),
]


@pytest.mark.parametrize("case", CASES, ids=["%s-b%d-c%d-%dx%d%s" % (c[4], c[0], c[1], c[2], c[3], "-cl" if c[5] else "") for c in CASES])
def test_bias_gradient(case):
    B, C, H, W, dtype, nhwc, shift = case
    say("bias gradient %s" % (case,))
    dY = synth.draw((B, C, H, W), 81, "normal", 1.0, dtype)
    flat = np.ascontiguousarray(dY.transpose(0, 2, 3, 1) if nhwc else dY).reshape(-1)
    t = torch.zeros(flat.size + 16, dtype=TD[dtype], device=DEV)
    t[shift:shift + flat.size] = xb.to_device(flat, dtype, DEV)
    d = xb.make_desc(B, 1, C, H, W, 1, 1, 0, 1, dtype, "rademacher", 1, xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
    db = torch.full((C,), float("nan"), dtype=TD[dtype], device=DEV)
    xb.xconv_bias_grad(d, t.data_ptr() + shift * t.element_size(), db, xb.alloc_bytes(xb.xconv_bias_workspace_bytes(d)))
    want = dY.astype(np.float64).sum(axis=(0, 2, 3))
    got = db.double().cpu().numpy()
    ulp = {"f32": 0.0, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dtype]
    bound = 1.01 * ulp * np.abs(want) + 1e-6 * np.abs(dY).astype(np.float64).sum(axis=(0, 2, 3))
    assert np.all(np.abs(got - want) <= bound), np.max(np.abs(got - want) - bound)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("C_out", [24, 1040], ids=["one-launch", "two-launches"])
def test_weight_gradient_in_the_weights_type(dtype, C_out):
    say("weight gradient in %s, %d channels" % (dtype, C_out))
    d = xb.make_desc(3, 40, C_out, 9, 8, 3, 1, 1, 16, dtype, "rademacher", 5)
    X = xb.to_device(synth.draw((3, 40, 9, 8), 82, "relu_normal", 1.0, dtype), dtype, DEV)
    dY = xb.to_device(synth.draw((3, C_out, 9, 8), 83, "normal", 1e-2, dtype), dtype, DEV)
    Xt = xb.alloc_xt(d)
    xb.xconv_probe_fwd(d, X, Xt, None, xb.alloc_ws(d, xb.XCONV_OP_PROBE))
    full = torch.empty((C_out, 40, 3, 3), dtype=torch.float32, device=DEV)
    short = torch.empty((C_out, 40, 3, 3), dtype=TD[dtype], device=DEV)
    ws = xb.alloc_ws(d, xb.XCONV_OP_ESTIMATE)
    xb.xconv_dw_estimate(d, dY, Xt, None, full, ws)
    xb.xconv_dw_estimate_as(d, dY, Xt, None, short, d.dtype, ws)
    assert torch.equal(full.to(TD[dtype]), short)
    xbar = torch.empty((3, 16), dtype=torch.float32, device=DEV)
    xb.xconv_pixel_probe_fwd(d, X, xbar, xb.alloc_bytes(xb.xconv_pixel_workspace_bytes(d, xb.XCONV_OP_PROBE)))
    ws = xb.alloc_bytes(xb.xconv_pixel_workspace_bytes(d, xb.XCONV_OP_ESTIMATE))
    xb.xconv_pixel_dw_estimate(d, dY, xbar, full, ws)
    xb.xconv_pixel_dw_estimate_as(d, dY, xbar, short, d.dtype, ws)
    assert torch.equal(full.to(TD[dtype]), short)
    d.keep_q15 = 16384
    with pytest.raises(xb.XConvError):
        xb.xconv_pixel_dw_estimate_as(d, dY, xbar, short, d.dtype, ws)
