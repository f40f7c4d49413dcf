"""Forward convolution and input gradient of layers at the limits of the kernels' 32-bit offsets: tiles that would cross many large
images (narrow strips of flattened 1x1 layers, few long rows), and images past a 2 GiB buffer descriptor (64-bit addresses).
Compared on windows of columns against double-precision convolutions of the same storage values."""
import pytest
import torch

from paper_2106_06998_amd import binding as xb
from test_gpu_conv import DEV, TD, check, say

pytestmark = pytest.mark.gpu

# B, C_in, C_out, H, W, k, pad, dtype, channels-last, 64-bit addresses
CASES = [
    (8, 256, 1024, 500, 500, 1, 0, "bf16", True, False),
    (8, 384, 192, 500, 500, 1, 0, "f32", True, False),
    (24, 128, 64, 3, 80000, 3, 1, "f16", False, False),
    (1, 1, 2, 11000, 11000, 3, 1, "f32", False, True),     # few channels of planes that fill a unit past 2 GiB
    (2, 3, 1, 12000, 12000, 3, 1, "f16", False, True),
    (1, 3, 2, 9001, 12001, 1, 0, "bf16", False, True),
    (2, 3, 5, 5500, 5500, 3, 1, "f16", False, False),      # just below
    (300, 2, 3, 2048, 2048, 3, 1, "f16", False, False),    # more positions than a launch counts: two runs of images
    (2, 64, 8, 4200, 4200, 3, 1, "f16", False, True),
    (2, 8, 64, 3000, 3000, 3, 1, "f32", True, True),
]


def windows(src, weight, image, cols, W, pad):
    """Convolution (pad rows and columns of zeros) of all rows and the columns `cols` of one image in double precision."""
    lo, hi = cols[0] - pad, cols[1] + pad
    x = src[image:image + 1, :, :, max(lo, 0):min(hi, W)].double().cpu()
    x = torch.nn.functional.pad(x, (max(-lo, 0), max(hi - W, 0), pad, pad))
    return torch.nn.functional.conv2d(x, weight)


@pytest.mark.parametrize("packed", [True, False], ids=["packed", "gathered"])
@pytest.mark.parametrize("case", CASES, ids=["%s%s-b%d-c%d-%d-%dx%d-k%d" % (c[7], "-cl" if c[8] else "", *c[:6]) for c in CASES])
def test_large_layers(case, packed):
    B, C_in, C_out, H, W, k, p, dtype, nhwc, big = case
    d = xb.make_desc(B, C_in, C_out, H, W, k, 1, p, 1, dtype, layout=xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
    fmt = torch.channels_last if nhwc else torch.contiguous_format
    g = torch.Generator(device=DEV).manual_seed(7)

    def tensor(shape, std, relu=False):
        # one image at a time: the draw itself is in fp32
        t = torch.empty(shape, dtype=TD[dtype], device=DEV, memory_format=fmt)
        for b in range(shape[0]):
            v = torch.randn(shape[1:], device=DEV, generator=g).mul_(std)
            t[b] = v.relu_() if relu else v
        return t

    w = (torch.randn((C_out, C_in, k, k), device=DEV, generator=g) / (C_in * k * k)).to(TD[dtype])
    w64 = w.double().cpu()
    for transposed, cin, cout in ((0, C_in, C_out), (1, C_out, C_in)):
        assert xb.xconv_conv_plan_info(d, transposed, packed)["big"] == big
        say("large %s: %s, packed %s" % ("input gradient" if transposed else "forward", case, packed))
        src = tensor((B, cin, H, W), 1e-2 if transposed else 1.0, not transposed)
        out = torch.full((B, cout, H, W), float("nan"), dtype=TD[dtype], device=DEV).contiguous(memory_format=fmt)
        ws = xb.alloc_bytes(xb.xconv_conv_workspace_bytes(d, transposed)) if packed else None
        if transposed:
            xb.xconv_dx_exact_ws(d, src, w, out, ws)
        else:
            xb.xconv_conv_fwd_ws(d, src, w, None, out, ws)
        torch.cuda.synchronize()
        wt = w64.flip(2, 3).transpose(0, 1).contiguous() if transposed else w64
        for b in range(B):
            assert not bool(torch.isnan(out[b]).any())
            if b % (1 + B // 3) and b not in (B - 1, 255, 256):      # (the two runs above meet at image 256)
                continue
            for c0 in (0, W // 2 - 5, W - 8):
                want = windows(src, wt, b, (c0, c0 + 8), W, p)
                check(out[b:b + 1, :, :, c0:c0 + 8].double().cpu().numpy(), want.numpy(), dtype)
        del src, out
