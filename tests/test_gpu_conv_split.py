"""Products of fp32 layers on packed weights, which run on the 16-bit matrix cores with every float as the sum of three bf16 numbers:
channels around the edges of units, k-steps and chunks, both layouts, strides; scales far from one; infinities and NaN."""
import pytest
import torch
import torch.nn.functional as F

from paper_2106_06998_amd import binding as xb

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def products(X, dY, W, stride, pad, nhwc):
    B, C_in, H, Wd = X.shape
    d = xb.make_desc(B, C_in, W.shape[0], H, Wd, tuple(W.shape[2:]), stride, pad, 1, "f32", "rademacher", 1,
                     layout=xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
    put = (lambda t: t.permute(0, 2, 3, 1).contiguous().to(DEV)) if nhwc else (lambda t: t.contiguous().to(DEV))
    back = (lambda t: t.permute(0, 3, 1, 2).cpu()) if nhwc else (lambda t: t.cpu())
    Xd, dYd, Wd_ = put(X), put(dY), W.to(DEV)
    Y, dX = torch.full_like(dYd, float("nan")), torch.full_like(Xd, float("nan"))
    ws = [xb.alloc_bytes(xb.xconv_conv_workspace_bytes(d, t), DEV) for t in (0, 1)]
    xb.xconv_conv_fwd_ws(d, Xd, Wd_, None, Y, ws[0])
    xb.xconv_dx_exact_ws(d, dYd, Wd_, dX, ws[1])
    torch.cuda.synchronize()
    return back(Y), back(dX)


def reference(X, dY, W, stride, pad):
    X, dY, W = X.double(), dY.double(), W.double()
    return F.conv2d(X, W, None, stride, pad), torch.nn.grad.conv2d_input(X.shape, W, dY, stride, pad)


# B, C_in, C_out, H, W, k, stride, pad, channels-last
CASES = [
    (2, 1, 1, 5, 4, 1, 1, 0, False),
    (3, 8, 9, 9, 7, 3, 1, 1, False),
    (2, 16, 17, 12, 33, 3, 1, 1, False),
    (2, 12, 20, 11, 10, 3, 2, 1, True),          # whole vectors of four channels, no whole units of eight
    (2, 31, 33, 8, 21, 2, 1, 0, False),
    (1, 33, 64, 17, 16, 5, 2, 2, True),
    (2, 64, 40, 20, 20, 3, 1, 1, False),
    (1, 129, 136, 9, 11, 3, 1, 1, True),         # more channels than a resident patch has
    (1, 161, 24, 30, 28, 1, 1, 0, False),
]


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -60, 2.0 ** 50])
@pytest.mark.parametrize("case", CASES, ids=["c%d-%d-%dx%d-k%d-s%d-%s" % (c[1], c[2], c[3], c[4], c[5], c[6], "cl" if c[8] else "planes") for c in CASES])
def test_split_products_against_64_bits(case, scale):
    B, C_in, C_out, H, W, k, stride, pad, nhwc = case
    g = torch.Generator().manual_seed(C_in + 100 * k)
    X = torch.randn((B, C_in, H, W), generator=g) * scale
    Wt = torch.randn((C_out, C_in, k, k), generator=g)
    dY = torch.randn((B, C_out, (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1), generator=g) * scale
    got, want = products(X, dY, Wt, stride, pad, nhwc), reference(X, dY, Wt, stride, pad)
    size = reference(X.abs(), dY.abs(), Wt.abs(), stride, pad)
    for a, b, s, channels in zip(got, want, size, (C_in, C_out)):
        # the terms left out are 3 * 2^-25 of each product; a matrix instruction rounds its sum of 16 products once or twice, by at
        # most 2^-24 of the terms so far, and the two sums are added and stored
        steps = k * k * -(-channels // 16)
        bound = (2 * steps + 8) * 2.0 ** -24 * s
        bad = (a.double() - b).abs() > bound
        assert not bool(bad.any()), (int(bad.sum()), float(((a.double() - b).abs() / bound.clamp_min(1e-300)).max()))


@pytest.mark.parametrize("nhwc", [False, True])
@pytest.mark.parametrize("channels", [20, 136])      # resident, in chunks
def test_split_products_keep_infinities_and_nan(channels, nhwc):
    g = torch.Generator().manual_seed(channels)
    X = torch.randn((2, channels, 12, 11), generator=g)
    Wt = torch.randn((24, channels, 3, 3), generator=g)
    inf, top = float("inf"), torch.finfo(torch.float32).max
    X[0, 3, 4, 4], X[0, 7, 9, 2], X[1, 17, 5, 5], X[1, channels - 1, 9, 9] = inf, -inf, float("nan"), inf
    X[0, 9, 0, 9] = top                               # bf16 rounds it to an infinity
    Wt[2, 3], Wt[3, 3], Wt[4, 7], Wt[5, 3] = 0.5, 0.0, -1.0, 1.0 + 2.0 ** -12      # exact in one piece; 0 * inf; pieces of both signs
    Wt[:, 9] *= 0.25                                   # (no product with `top` overflows)
    Wt[12] *= 0.1
    Wt[8, channels - 1, 1, 1], Wt[9, 3, 1, 1], Wt[10, 2, 1, 1] = -inf, inf, float("nan")     # (the middle tap meets no padding)
    dY = torch.randn((2, 24, 12, 11), generator=g)
    dY[0, 11, 3, 3], dY[1, 12, 8, 8] = inf, top
    for a, b in zip(products(X, dY, Wt, 1, 1, nhwc), reference(X, dY, Wt, 1, 1)):
        b = b.float()
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isinf(a), torch.isinf(b))
        assert torch.equal(a[torch.isinf(b)], b[torch.isinf(b)])
        ok = torch.isfinite(b)
        assert bool(torch.isfinite(a[ok]).all()) and float(((a - b)[ok].abs() / (b[ok].abs() + 1)).max()) < 1e-5
