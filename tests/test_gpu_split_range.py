"""fp32 products and correlations on the 16-bit matrix cores over the whole range of a float: values near the smallest normal one and
below it, sums of one or two products, sums that come out next to the largest one, factors of very different size, an infinity beside the smallest numbers.  What the pieces of
a split float do not hold has to come out as the fp32 matrix instructions give it."""
import pytest
import torch

from paper_2106_06998_amd import binding as xb
from test_gpu_conv_split import products, reference
from test_gpu_corr_split import split_taken, weight_gradient

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LAST = 2.0 ** -149                                                  # the last place of a subnormal number

# C_in, C_out, H, W, k, stride, channels-last: resident and in chunks, one and two blocks of positions a wave, classes of positions
PRODUCTS = [(24, 40, 13, 12, 3, 1, False), (24, 40, 12, 13, 3, 2, False), (136, 33, 9, 11, 3, 1, True), (160, 64, 40, 40, 1, 1, False), (7, 9, 6, 5, 1, 1, True)]
# log2 of the scale of the data and of the weights; their product stays within the normal numbers, or rounds to subnormal ones
SCALES = [(-112, 0), (-124, 0), (0, -118), (-100, 90), (118, -120), (-120, 118), (-64, -64), (55, 55)]


def drawn(shape, g, e):
    return (torch.randn(shape, generator=g, dtype=torch.float64) * 2.0 ** e).float()


@pytest.mark.parametrize("scales", SCALES, ids=["2^%d*2^%d" % s for s in SCALES])
@pytest.mark.parametrize("case", PRODUCTS, ids=["c%d-%d-%dx%d-k%d-s%d-%s" % (*c[:6], "cl" if c[6] else "planes") for c in PRODUCTS])
def test_products_at_all_magnitudes(case, scales):
    C_in, C_out, H, W, k, stride, nhwc = case
    g = torch.Generator().manual_seed(C_in)
    pad = k // 2
    X, Wt = drawn((2, C_in, H, W), g, scales[0]), drawn((C_out, C_in, k, k), g, scales[1])
    dY = drawn((2, C_out, (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1), g, scales[0])
    got, want = products(X, dY, Wt, stride, pad, nhwc), reference(X, dY, Wt, stride, pad)
    size = reference(X.abs(), dY.abs(), Wt.abs(), stride, pad)
    for a, b, s, channels in zip(got, want, size, (C_in, C_out)):
        # split: sums of 16 products that round once or twice (test_gpu_conv_split.py); fp32 instructions: two products at a time, each
        # rounded.  Subnormal sums round to whole last places, and so may each partial sum
        terms = k * k * channels
        bound = (terms + 8) * (2.0 ** -24 * s + (LAST if scales[0] + scales[1] < -100 else 0))
        assert bool(((a.double() - b).abs() <= bound).all()), float(((a.double() - b).abs() / bound).max())


@pytest.mark.parametrize("channels", [1, 2])
@pytest.mark.parametrize("k, stride", [(1, 1), (3, 2)])      # (strided: positions with one and two of the nine taps)
def test_sums_of_one_and_two_products_are_those_of_fp32(channels, k, stride):
    # one or two roundings, and none for what a product leaves out
    g = torch.Generator().manual_seed(channels)
    X, Wt = drawn((3, channels, 24, 20), g, 0), drawn((channels, channels, k, k), g, 0)
    dY = drawn((3, channels, 24 // stride, 20 // stride), g, 0)
    got, want = products(X, dY, Wt, stride, k // 2, False), reference(X, dY, Wt, stride, k // 2)
    size = reference(X.abs(), dY.abs(), Wt.abs(), stride, k // 2)
    if k == 1:
        assert bool(((got[0].double() - want[0]).abs() <= channels * 2.0 ** -24 * size[0]).all())
    one_tap = (got[1].double() - want[1], size[1]) if k == 1 else ((got[1].double() - want[1])[:, :, ::2, ::2], size[1][:, :, ::2, ::2])
    assert bool((one_tap[0].abs() <= channels * 2.0 ** -24 * one_tap[1]).all())


@pytest.mark.parametrize("side", ["data", "weights", "sum"])
def test_products_next_to_the_largest_float(side):
    X, Wt = torch.zeros((1, 8, 4, 4)), torch.zeros((32, 8, 1, 1))
    dY = torch.zeros((1, 32, 4, 4))
    x, w = {"data": (1.9995 * 2.0 ** 127, 1.0), "weights": (0.998, 1.9995 * 2.0 ** 127), "sum": (1.998 * 2.0 ** 63, 1.9995 * 2.0 ** 63)}[side]
    X[0, 3, 1, 2], dY[0, 5, 2, 1], Wt[5, 3] = x, x, w
    X[0, 2, 3, 3], dY[0, 6, 3, 3], Wt[6, 2] = 3.0, 3.0, 0.1          # untouched by it, in the same tile
    for a, b in zip(products(X, dY, Wt, 1, 0, False), reference(X, dY, Wt, 1, 0)):
        assert float(b.abs().max()) < 3.4028e38 and torch.equal(a, b.float())


@pytest.mark.parametrize("tiny", [2.0 ** -126, 1.5 * 2.0 ** -140, LAST])
def test_an_infinity_times_the_smallest_numbers(tiny):
    inf = float("inf")
    X, Wt, dY = torch.zeros((1, 8, 4, 4)), torch.full((16, 8, 1, 1), tiny), torch.zeros((1, 16, 4, 4))
    X[0, 3, 1, 2], dY[0, 5, 2, 1] = inf, -inf
    X[0, :, 3, 3], dY[0, :, 0, 0] = tiny, -tiny
    for a, b in zip(products(X, dY, Wt, 1, 0, False), reference(X, dY, Wt, 1, 0)):
        assert torch.equal(a, b.float())
    Wt.fill_(inf)
    X.masked_fill_(X != 0, tiny), dY.masked_fill_(dY != 0, -tiny)
    for a, b in zip(products(X, dY, Wt, 1, 0, False), reference(X, dY, Wt, 1, 0)):
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(a.nan_to_num(1.0), b.float().nan_to_num(1.0))


@pytest.mark.parametrize("nhwc", [False, True])
def test_the_bias_is_added_to_sums_that_are_computed_again(nhwc):
    # one product a sum, and sums on either side that the pieces hold
    g = torch.Generator().manual_seed(5)
    X, Wt, bias = torch.zeros((2, 16, 6, 10)), torch.zeros((40, 16, 1, 1)), torch.randn(40, generator=g) * 2.0 ** 84
    Wt[torch.arange(40), torch.arange(40) % 16] = torch.randn(40, generator=g).view(40, 1, 1)
    X[:, 3], X[1, 7, 2, 4], X[0, 9, 5, 9] = 1.5 * 2.0 ** 105, float("inf"), float("nan")
    X[:, 10] = torch.randn((2, 6, 10), generator=g)
    d = xb.make_desc(2, 16, 40, 6, 10, 1, 1, 0, 1, "f32", "rademacher", 1, layout=xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
    Xd = (X.permute(0, 2, 3, 1) if nhwc else X).contiguous().to(DEV)
    Y = torch.full((2, 6, 10, 40) if nhwc else (2, 40, 6, 10), float("nan"), device=DEV)
    xb.xconv_conv_fwd_ws(d, Xd, Wt.to(DEV), bias.to(DEV), Y, xb.alloc_bytes(xb.xconv_conv_workspace_bytes(d, 0), DEV))
    torch.cuda.synchronize()
    got = (Y.permute(0, 3, 1, 2) if nhwc else Y).cpu()
    want = torch.nn.functional.conv2d(X.double(), Wt.double()).float() + bias.view(1, 40, 1, 1)
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    finite = torch.isfinite(want)
    assert torch.equal(got[~finite].nan_to_num(0.0), want[~finite].nan_to_num(0.0))
    assert bool(((got - want)[finite].abs() <= 2.0 ** -23 * (want - bias.view(1, 40, 1, 1))[finite].abs() + 2.0 ** -23 * want[finite].abs()).all())


# B, C_in, C_out, H, W, k, stride, splits: 16 columns side by side and 32, four, two and one waves along the reduction, a narrow last
# strip, several runs, strides beside and beyond the kernel's rows
CORRELATIONS = [(9, 48, 72, 10, 28, 3, 1, 3), (8, 40, 30, 24, 20, 5, 1, 1), (6, 64, 24, 11, 36, 3, 1, 2), (16, 96, 64, 12, 24, 3, 2, 3), (9, 32, 40, 23, 23, 3, 3, 1)]


def exact_gradient(case, X, dY, monkeypatch):
    B, C_in, C_out, H, W, k, s, splits = case
    monkeypatch.setenv("XCONV_WS32_SPLITS", str(splits))
    d = xb.make_desc(B, C_in, C_out, H, W, k, s, k // 2, 8, "f32", "rademacher", 7)
    assert split_taken(d, xb.XCONV_OP_EXACT)
    dw = torch.full((C_out, C_in, k, k), float("nan"), device=DEV)
    xb.xconv_dw_exact(d, dY.to(DEV), X.to(DEV), dw, xb.alloc_ws(d, xb.XCONV_OP_EXACT, DEV))
    torch.cuda.synchronize()
    return dw.cpu()


def correlation_data(case, g, ex, ey):
    B, C_in, C_out, H, W, k, s, _ = case
    p = k // 2
    return drawn((B, C_in, H, W), g, ex), drawn((B, C_out, (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1), g, ey)


@pytest.mark.parametrize("scales", SCALES, ids=["2^%d*2^%d" % s for s in SCALES])
@pytest.mark.parametrize("case", CORRELATIONS, ids=["b%d-c%d-%d-%dx%d-k%d-s%d" % c[:7] for c in CORRELATIONS])
def test_correlations_at_all_magnitudes(case, scales, monkeypatch):
    X, dY = correlation_data(case, torch.Generator().manual_seed(case[0]), *scales)
    k, s = case[5:7]
    got = exact_gradient(case, X, dY, monkeypatch)
    want, size = (weight_gradient(a, b, (k, k), s, k // 2) for a, b in ((X, dY), (X.abs(), dY.abs())))
    # as many roundings as terms at the worst, and a tenth of that: terms of random signs come nowhere near
    terms = case[0] * dY.shape[2] * dY.shape[3]
    bound = (0.1 * terms + 8) * (2.0 ** -24 * size + (LAST if sum(scales) < -100 else 0))
    assert bool(((got.double() - want).abs() <= bound).all()), float(((got.double() - want).abs() / bound).max())


@pytest.mark.parametrize("case", CORRELATIONS, ids=["b%d-c%d-%d-%dx%d-k%d-s%d" % c[:7] for c in CORRELATIONS])
def test_correlations_of_infinities_and_the_largest_floats(case, monkeypatch):
    g = torch.Generator().manual_seed(case[1])
    X, dY = correlation_data(case, g, 0, 0)
    k, s = case[5:7]
    inf = float("inf")
    X[:, 3:12] = 0
    dY[:, 2:9] = 0
    y, x = 4, 4                                     # an output pixel; its middle input pixel
    X[1, 3, y * s, x * s], dY[1, 2, y, x] = 1.998 * 2.0 ** 63, 1.9995 * 2.0 ** 63        # next to the largest float
    X[2, 4, y * s, x * s], dY[2, 3, y, x] = 1.9995 * 2.0 ** 127, 0.5
    X[3, 5, y * s, x * s], dY[3, 4, y, x] = 2.0 ** -149, inf                              # an infinity and the smallest number
    X[4, 6, y * s, x * s], dY[4, 5, y, x] = 2.0 ** 120, 2.0 ** -126
    X[5, 15, y * s, x * s] = -inf
    dY[0, 9, y, x] = float("nan")
    got, want = exact_gradient(case, X, dY, monkeypatch), weight_gradient(X, dY, (k, k), s, k // 2)
    assert float(want[2, 3, k // 2, k // 2]) > 3.39e38 and float(want[4, 5, k // 2, k // 2]) == inf
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    largest = float(torch.finfo(torch.float32).max)
    assert torch.equal(got.clamp(-largest, largest)[want.abs() > largest], want.float().clamp(-largest, largest)[want.abs() > largest])
    ok = want.abs() <= largest                      # (NaN and beyond the largest float: above)
    size = weight_gradient(X.abs().nan_to_num(0, 0, 0), dY.abs().nan_to_num(0, 0, 0), (k, k), s, k // 2)
    terms = case[0] * dY.shape[2] * dY.shape[3]
    assert bool(((got.double() - want).abs() <= (0.1 * terms + 8) * (2.0 ** -24 * size + LAST))[ok].all())
