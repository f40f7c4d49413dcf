"""Every one of the six products of split floats counts: sums of few terms on the 16-bit matrix cores against 64 bits, with a bound that
the same sums without the third pieces, or without the product of the second ones, exceed (computed here in 64 bits).  Correlations with 16
columns side by side and 32, one and two blocks of output channels, strides up to and beyond the kernel's rows."""
import pytest
import torch

from paper_2106_06998_amd import binding as xb
from test_gpu_conv_split import products, reference
from test_gpu_corr_split import split_taken, weight_gradient

DEV = "cuda:0"
KEPT = [(2, 0), (0, 2), (1, 1), (1, 0), (0, 1), (0, 0)]


def pieces(x):
    out, rest = [], x
    for _ in range(3):
        out.append(rest.bfloat16().float())
        rest = rest - out[-1]
    assert not bool(rest.any())
    return [p.double() for p in out]


def bound(terms):
    # a sum of 16 products rounds once or twice, each time by 2^-24 * 0.58 (the root mean square of a rounding, at the worst place between
    # two powers of two) of a sum that grows like the root of its terms; storing, adding the two sums and what a product leaves out: one more
    return 2.0 ** -24 * (0.58 * (-(-terms // 16)) ** 0.5 + 1)


def norm_error(got, want):
    return float((got - want).norm() / want.norm())


def without(op, a, b, left_out):
    A, B = pieces(a), pieces(b)
    return sum(op(A[i], B[j]) for i, j in KEPT if not left_out(i, j))


MISTAKES = {"third pieces": lambda i, j: 2 in (i, j), "second pieces' product": lambda i, j: (i, j) == (1, 1)}

# B, C_in, C_out, H, W, kernel, stride, pad
CORRELATIONS = [
    (5, 48, 72, 6, 8, (3, 3), 1, (1, 1)),
    (5, 48, 24, 6, 8, (3, 3), 1, (1, 1)),
    (6, 64, 72, 5, 12, (3, 3), 1, (1, 1)),
    (6, 64, 24, 5, 12, (3, 3), 1, (1, 1)),
    (8, 32, 40, 12, 24, (3, 3), 3, (0, 1)),
    (8, 48, 40, 14, 25, (2, 4), 3, (0, 0)),          # rows of A that no step reads
    (7, 32, 33, 9, 15, (3, 3), 2, (1, 1)),
]
IDS = ["b%d-c%d-%d-%dx%d-k%dx%d-s%d" % (*c[:5], *c[5], c[6]) for c in CORRELATIONS]


def correlation(case):
    B, C_in, C_out, H, W, k, s, p = case
    g = torch.Generator().manual_seed(C_in + C_out)
    X = torch.randn((B, C_in, H, W), generator=g)
    dY = torch.randn((B, C_out, (H + 2 * p[0] - k[0]) // s + 1, (W + 2 * p[1] - k[1]) // s + 1), generator=g)
    return X, dY, bound(B * dY.shape[2] * dY.shape[3]), lambda a, b: weight_gradient(a, b, k, s, p)


@pytest.mark.gpu
@pytest.mark.parametrize("splits", ["1", "2"])
@pytest.mark.parametrize("case", CORRELATIONS, ids=IDS)
def test_correlations_of_few_terms(case, splits, monkeypatch):
    monkeypatch.setenv("XCONV_WS32_SPLITS", splits)
    B, C_in, C_out, H, W, k, s, p = case
    d = xb.make_desc(B, C_in, C_out, H, W, k, (s, s), p, 8, "f32", "rademacher", 7)
    assert split_taken(d, xb.XCONV_OP_EXACT)
    X, dY, limit, op = correlation(case)
    dw = torch.full((C_out, C_in, *k), float("nan"), device=DEV)
    xb.xconv_dw_exact(d, dY.to(DEV), X.to(DEV), dw, xb.alloc_ws(d, xb.XCONV_OP_EXACT, DEV))
    torch.cuda.synchronize()
    assert norm_error(dw.cpu().double(), op(X, dY)) <= limit


@pytest.mark.parametrize("mistake", MISTAKES)
@pytest.mark.parametrize("case", CORRELATIONS, ids=IDS)
def test_the_bound_of_correlations_shows_a_product_left_out(case, mistake):
    X, dY, limit, op = correlation(case)
    assert norm_error(without(op, X, dY, MISTAKES[mistake]), op(X, dY)) > limit


# C_in, C_out, kernel, channels-last: both products; resident and in chunks (more than 128 channels)
PRODUCTS = [(9, 16, 1, False), (16, 12, 1, True), (24, 33, 3, False), (136, 40, 1, False), (136, 136, 1, True)]


def product(case):
    C_in, C_out, k, _ = case
    g = torch.Generator().manual_seed(C_in)
    return torch.randn((2, C_in, 11, 10), generator=g), torch.randn((2, C_out, 11, 10), generator=g), torch.randn((C_out, C_in, k, k), generator=g)


@pytest.mark.gpu
@pytest.mark.parametrize("case", PRODUCTS, ids=["c%d-%d-k%d-%s" % (*c[:3], "cl" if c[3] else "planes") for c in PRODUCTS])
def test_products_of_few_terms(case):
    C_in, C_out, k, nhwc = case
    X, dY, W = product(case)
    for got, want, channels in zip(products(X, dY, W, 1, k // 2, nhwc), reference(X, dY, W, 1, k // 2), (C_in, C_out)):
        assert norm_error(got.double(), want) <= bound(k * k * -(-channels // 16) * 16)


@pytest.mark.parametrize("mistake", MISTAKES)
@pytest.mark.parametrize("case", PRODUCTS, ids=["c%d-%d-k%d-%s" % (*c[:3], "cl" if c[3] else "planes") for c in PRODUCTS])
def test_the_bound_of_products_shows_a_product_left_out(case, mistake):
    C_in, C_out, k, _ = case
    X, dY, W = product(case)
    want = reference(X, dY, W, 1, k // 2)
    forward = without(lambda a, b: reference(a, dY, b, 1, k // 2)[0], X, W, MISTAKES[mistake])
    backward = without(lambda a, b: reference(X, a, b, 1, k // 2)[1], dY, W, MISTAKES[mistake])
    for got, exact, channels in zip((forward, backward), want, (C_in, C_out)):
        assert norm_error(got, exact) > bound(k * k * -(-channels // 16) * 16)
