"""The convolution kernels at the edges of their tiles, against the oracle: every wave shape, both ways the weights are read
(packed into a workspace, gathered from W), patches
resident and in chunks, the three ways the input patch is read (pairs of columns, whole channel units,
single elements), ragged channels and positions, tiles over several images, strided input gradients with classes of one,
several and no taps, patches too large for a full tile, and the bias (added to the rounded product)."""
import numpy as np
import pytest
import torch

from oracle import xconv_oracle as xo
from paper_2106_06998_amd import binding as xb
from paper_2106_06998_amd import synth
from test_gpu_conv import DEV, TD, check, say

pytestmark = pytest.mark.gpu

# B, C_in, C_out, H, W, k, stride, pad, dtype, channels-last
CASES = [
    (5, 16, 33, 7, 7, 3, 1, 1, "f32", False),        # tiles over several images
    (2, 40, 100, 9, 34, 3, 1, 1, "f16", False),      # pairs of columns, second k-step of the last chunk empty
    (3, 33, 65, 5, 13, 3, 1, 1, "bf16", False),      # odd width: single elements
    (2, 48, 40, 6, 18, 3, 2, 1, "f16", False),       # columns split by the stride
    (2, 24, 72, 11, 9, 5, 2, 2, "bf16", True),       # whole channel units, channels-last output
    (2, 12, 20, 10, 10, 1, 2, 0, "f32", True),       # input gradient: classes without taps
    (2, 9, 17, 15, 14, 3, 3, 0, "f16", True),        # channels that are no whole units
    (3, 8, 8, 21, 14, 7, 7, 0, "f16", False),        # a stride as large as the kernel
    (2, 24, 16, 19, 22, 3, 5, 1, "bf16", False),     # more classes without taps than with
    (3, 16, 9, 17, 30, 1, 8, 0, "f16", False),
    (2, 12, 10, 13, 11, 5, 5, 2, "f32", True),       # more classes than a launch takes
    (2, 4, 6, 1, 1, 1, 5, 2, "f16", False),          # an output that reads the padding only: no class has taps
    (40, 16, 16, 1, 1, (7, 1), 1, (3, 0), "f32", False),   # one position per image
    (1, 64, 32, 3, 300, 3, 1, 1, "bf16", False),     # strips of a wide row
    (2, 150, 136, 8, 10, 3, 1, 1, "f16", False),     # more channels than a resident patch: chunks
    (2, 133, 40, 9, 7, 3, 2, 1, "f32", False),
    (1, 168, 200, 7, 6, 3, 1, 1, "bf16", True),
]


# weights gathered for one, two and four waves of 32 output channels: groups of 8, 4 and 2 k-steps that kernel offsets and channels
# do not fill evenly
GATHERS = [
    (2, 150, 136, 8, 10, 3, 1, 1, "f16", False),
    (1, 168, 200, 7, 6, 3, 1, 1, "bf16", True),
    (2, 133, 70, 9, 7, 3, 2, 1, "f32", False),
    (3, 68, 72, 5, 9, (1, 5), 1, (0, 2), "f32", True),
    (2, 100, 66, 6, 8, 1, 1, 0, "bf16", False),
]


@pytest.mark.parametrize("waves", ["1", "2", "4"])
@pytest.mark.parametrize("case", GATHERS, ids=["%s-c%d-%d-k%s-s%s" % (c[8], c[1], c[2], c[5], c[6]) for c in GATHERS])
def test_gathered_weights_of_several_waves(case, waves, monkeypatch):
    monkeypatch.setenv("XCONV_CONV_WM", waves)
    run_tiles(case, False, "11", monkeypatch)


@pytest.mark.parametrize("shape", ["0", "24", "22", "12", "11"])
@pytest.mark.parametrize("packed", [True, False], ids=["packed", "gathered"])
@pytest.mark.parametrize("case", CASES, ids=["%s-c%d-%d-k%s-s%s" % (c[8], c[1], c[2], c[5], c[6]) for c in CASES])
def test_conv_tiles(case, packed, shape, monkeypatch):
    run_tiles(case, packed, shape, monkeypatch)


# classes of unequal size take turns in the grid: a tile past the last of its class does nothing.  Classes of one tile each, then rows
# of 2 and 1 times 1501 and 1500 positions (151 and 150), which no tile holds: the smallest class has about half of the largest's tiles
UNEQUAL = [
    (3, 16, 24, 1, 5, 3, 2, 1, "bf16", False),
    (2, 40, 16, 3, 301, 5, 2, 2, "f32", False),
    (1, 24, 40, 33, 2, 3, 2, 1, "f16", True),
    (4, 144, 24, 5, 3, 3, 2, 1, "f16", False),
    (1, 24, 16, 3, 3001, 3, 2, 1, "bf16", False),
    (1, 24, 40, 3, 3001, 3, 2, 1, "f16", True),
    (1, 24, 144, 3, 3001, 3, 2, 1, "f16", False),    # the contraction over 144 channels in chunks
]


@pytest.mark.parametrize("packed", [True, False], ids=["packed", "gathered"])
@pytest.mark.parametrize("case", UNEQUAL, ids=["%s-%dx%d" % (c[8], c[3], c[4]) for c in UNEQUAL])
def test_classes_of_unequal_size(case, packed, monkeypatch):
    B, C_in, C_out, H, W, k, s, p, dtype, nhwc = case
    if W >= 301:
        d = xb.make_desc(B, C_in, C_out, H, W, k, s, p, 1, dtype, "rademacher", 1, layout=xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
        v = xb.xconv_conv_plan_info(d, 1, packed)
        tile = 32 * (v["shape"] % 10) * (4 // v["WM"])
        # 2 x 1501 positions have more tiles than 1 x 1500, also with one tile lost to the end of a strip
        assert (v["launches"], v["classes"]) == (1, 4) and -(-2 * ((W + 1) // 2) // tile) > -(-(W // 2) // tile) + (W > 301)
        assert C_out < 144 or not v["res"]
    run_tiles(case, packed, "0", monkeypatch)


def run_tiles(case, packed, shape, monkeypatch):
    B, C_in, C_out, H, W, k, s, p, dtype, nhwc = case
    monkeypatch.setenv("XCONV_CONV_SHAPE", shape)
    (kH, kW), (ph, pw) = (k, k) if isinstance(k, int) else k, (p, p) if isinstance(p, int) else p
    say("conv tiles: %s packed %s shape %s" % (case, packed, shape))
    Ho, Wo = xo.out_extent(H, kH, s, ph), xo.out_extent(W, kW, s, pw)
    X = synth.draw((B, C_in, H, W), 71, "relu_normal", 1.0, dtype)
    dY = synth.draw((B, C_out, Ho, Wo), 72, "normal", 1e-2, dtype)
    Wt = synth.draw((C_out, C_in, kH, kW), 73, "normal", 1.0 / (C_in * kH * kW), dtype)
    bias = synth.draw((C_out,), 74, "normal", 1.0, dtype)
    d = xb.make_desc(B, C_in, C_out, H, W, (kH, kW), s, (ph, pw), 1, dtype, "rademacher", 1, layout=xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
    perm, back = ((0, 2, 3, 1), (0, 3, 1, 2)) if nhwc else ((0, 1, 2, 3), (0, 1, 2, 3))
    Xd, dYd = (xb.to_device(np.ascontiguousarray(t.transpose(perm)), dtype, DEV) for t in (X, dY))
    Wd, bd = xb.to_device(Wt, dtype, DEV), xb.to_device(bias, dtype, DEV)
    outs = []
    for b in (None, bd):
        Y = torch.full(tuple(np.array((B, C_out, Ho, Wo))[list(perm)]), float("nan"), dtype=TD[dtype], device=DEV)
        xb.xconv_conv_fwd_ws(d, Xd, Wd, b, Y, xb.alloc_bytes(xb.xconv_conv_workspace_bytes(d, 0)) if packed else None)
        outs.append(Y)
    dX = torch.full(tuple(np.array((B, C_in, H, W))[list(perm)]), float("nan"), dtype=TD[dtype], device=DEV)
    xb.xconv_dx_exact_ws(d, dYd, Wd, dX, xb.alloc_bytes(xb.xconv_conv_workspace_bytes(d, 1)) if packed else None)
    torch.cuda.synchronize()
    host = [t.float().cpu().numpy().transpose(back).astype(np.float64) for t in (*outs, dX)]
    assert all(np.all(np.isfinite(t)) for t in host)
    check(host[0], xo.conv_fwd(X, Wt.astype(np.float64), (s, s), (ph, pw)), dtype)
    check(host[2], xo.dx(dY, Wt.astype(np.float64), H, W, (s, s), (ph, pw)), dtype)
    b4 = bd.view(1, 1, 1, -1) if nhwc else bd.view(1, -1, 1, 1)
    assert torch.equal(outs[1], outs[0] + b4)


def test_conv_workspace_must_be_large_enough():
    d = xb.make_desc(2, 8, 8, 8, 8, 3, 1, 1, 1, "f32", "rademacher", 1)
    t = torch.zeros(4096, dtype=torch.float32, device=DEV)
    L, n = xb.lib(), xb.xconv_conv_workspace_bytes(d, 0)
    p = t.data_ptr()
    assert n > 0 and L.xconv_conv_fwd_ws(xb.ctypes.byref(d), p, p, None, p, p, n - 1, None) == xb.XCONV_EWORKSPACE
    assert L.xconv_dx_exact_ws(xb.ctypes.byref(d), p, p, p, p + 4, 1 << 20, None) == xb.XCONV_EINVAL
