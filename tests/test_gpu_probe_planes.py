"""The probe on planes of a ragged number of pixels (and volumes with such depth slices): a plane's last group of pixels is
moved back to end with it and overlaps the one before.  Every pixel against the oracle, repeated calls bit for bit."""
import numpy as np
import pytest
import torch

from oracle import xconv_oracle as xo
from paper_2106_06998_amd import binding as xb
from paper_2106_06998_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# storage rounding of the result plus fp32 sums of at most 72 products
TOL = {"f32": 1e-5, "f16": 2e-3, "bf16": 1e-2}


# planes below, at and just above the groups of 4 and 8 pixels, and with a remainder of one, two and three
@pytest.mark.parametrize("hw", [(1, 3), (2, 2), (1, 5), (7, 1), (1, 9), (2, 5), (7, 7), (3, 37), (45, 57)])
@pytest.mark.parametrize("dtype,probe,C,r", [("f32", "gaussian", 24, 12), ("f32", "rademacher", 33, 40), ("bf16", "rademacher", 40, 16),
                                             ("bf16", "gaussian", 17, 8), ("f16", "rademacher", 72, 36), ("f16", "gaussian", 33, 64)])
def test_ragged_planes(hw, dtype, probe, C, r):
    (H, W), B = hw, 5
    X = synth.draw((B, C, H, W), 31, "relu_normal", 1.0, dtype)
    d = xb.make_desc(B, C, 8, H, W, 1, 1, 0, r, dtype, probe, 77)
    Xd = xb.to_device(X, dtype, DEV)
    outs = []
    for _ in range(2):
        Xt = xb.alloc_xt(d, DEV)
        Xt.fill_(0x7f)
        xb.xconv_probe_fwd(d, Xd, Xt, None, xb.alloc_ws(d, xb.XCONV_OP_PROBE, DEV))
        out = torch.empty((B, r, H, W), dtype=torch.float32, device=DEV)
        xb.xconv_xt_unpack(d, Xt, out)
        torch.cuda.synchronize()
        outs.append((Xt, out.cpu().numpy()))
    assert torch.equal(outs[0][0], outs[1][0])
    dist, dt = (xo.GAUSSIAN if probe == "gaussian" else xo.RADEMACHER), {"f32": xo.F32, "bf16": xo.BF16, "f16": xo.F16}[dtype]
    want = xo.probe_fwd(X, xo.probe_matrix(dist, 77, C, r), dt)
    assert np.max(np.abs(outs[0][1] - want)) <= TOL[dtype] * np.max(np.abs(want))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dims", [(3, 1, 5), (4, 3, 3), (2, 5, 7)])
def test_ragged_depth_slices(dims, dtype):
    B, C, r = 2, 20, 8
    X, _ = synth.make_volume(B, C, 8, dims, dims, (41, 42, 43), dtype)
    d = xb.make_desc3d(B, C, 8, *dims, 3, 1, 1, r, dtype, "rademacher", 43)
    Xt = xb.alloc_bytes(xb.xconv3d_xt_bytes(d), DEV)
    xb.xconv3d_probe_fwd(d, xb.to_device(X, dtype, DEV), Xt, None, xb.alloc_bytes(xb.xconv3d_workspace_bytes(d, xb.XCONV_OP_PROBE), DEV))
    out = torch.empty((B, r, *dims), dtype=torch.float32, device=DEV)
    xb.xconv3d_xt_unpack(d, Xt, out)
    torch.cuda.synchronize()
    want = xo.probe_fwd3d(X, xo.probe_matrix(xo.RADEMACHER, 43, C, r), {"f32": xo.F32, "bf16": xo.BF16}[dtype])
    assert np.max(np.abs(out.cpu().numpy() - want)) <= TOL[dtype] * np.max(np.abs(want))


UNIT = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}     # largest relative error of rounding to the storage type


def probe_with(Z, C, hw, dtype, probe, X, with_ws):
    """Stored probe output of the given fp32 Z, as fp32 [B, r, H, W]."""
    (H, W), (B, r) = hw, (X.shape[0], Z.shape[1])
    d = xb.make_desc(B, C, 8, H, W, 1, 1, 0, r, dtype, probe, 5)
    Xt = xb.alloc_xt(d, DEV)
    out = torch.empty((B, r, H, W), dtype=torch.float32, device=DEV)
    xb.xconv_probe_fwd(d, xb.to_device(X, dtype, DEV), Xt, torch.from_numpy(Z).to(DEV), xb.alloc_ws(d, xb.XCONV_OP_PROBE, DEV) if with_ws else None)
    xb.xconv_xt_unpack(d, Xt, out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


# On ragged planes of 16-bit storage a given Z counts with all its fp32 bits, whatever the desc says of a Z that is drawn.  One channel:
# the product is rounded to fp32 and that to the storage type, and nothing else.
@pytest.mark.parametrize("with_ws", [True, False], ids=["scratch", "gathered"])
@pytest.mark.parametrize("probe", ["user", "rademacher"])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("hw,r", [((7, 7), 36), ((1, 5), 80), ((3, 37), 12)])
def test_given_z_keeps_its_bits(hw, r, dtype, probe, with_ws):
    X = synth.draw((40, 1) + hw, 61, "normal", 1.0, dtype)
    Z = synth.draw((1, r), 62, "normal", 1.0, "f32")
    want = synth.round_to_storage(Z.reshape(1, r, 1, 1) * X, dtype)
    assert np.array_equal(probe_with(Z, 1, hw, dtype, probe, X, with_ws), want)


# ... and with the range of fp32: entries that the storage type has no value or few bits for.  The sums of 40 products are at most
# 40 fp32 roundings of the sum of their sizes off, then rounded to the storage type.
@pytest.mark.parametrize("hw", [(7, 7), (1, 5), (3, 37)])
@pytest.mark.parametrize("dtype,zscale,xscale", [("f16", 1e6, 1e-5), ("f16", 1e-6, 1e3), ("bf16", 1e30, 1e-30), ("bf16", 1e-30, 1e30), ("f16", 1.0, 1e-7)])
def test_given_z_of_any_size(hw, dtype, zscale, xscale):
    C, r = 40, 20
    X = synth.draw((4, C) + hw, 63, "normal", xscale ** 2, dtype)
    Z = (synth.draw((C, r), 64, "normal", 1.0, "f32") * zscale).astype(np.float32)
    X64 = np.asarray(X, np.float64)
    want = np.einsum("nj,bnhw->bjhw", Z.astype(np.float64), X64)
    size = np.einsum("nj,bnhw->bjhw", np.abs(Z).astype(np.float64), np.abs(X64))
    got = probe_with(Z, C, hw, dtype, "user", X, True)
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - want) <= UNIT[dtype] * np.abs(want) + C * 2.0 ** -24 * size + (2.0 ** -25 if dtype == "f16" else 0))


# the projections of the pixel-probe estimators are such a Z for the planes of dY: beyond the range of f16 while the products are inside it
@pytest.mark.parametrize("dims", [(5, 7, 7, 9), (3, 5, 5, 5)])
def test_projections_beyond_half_precision(dims):
    C_in, C_out, H, W = dims
    B, r, k = 9, 12, 3
    d = xb.make_desc(B, C_in, C_out, H, W, k, 1, 0, r, "f16", "rademacher", 71)
    assert C_out * (H - 2) * (W - 2) % 4 != 0
    dY = synth.draw((B, C_out, H - 2, W - 2), 72, "normal", 1e-6, "f16")
    Z = xo.pixel_probe_matrix(xo.RADEMACHER, 71, C_in, H, W, r, xo.F16, 0)
    xbar = (synth.draw((B, r), 73, "normal", 1.0, "f32") * 1e6).astype(np.float32)
    want = xo.pixel_dw_estimate(dY, xbar, Z, C_in, H, W, k, k, (1, 1), (0, 0), nnz_norm=False)
    dW = torch.full((C_out, C_in, k, k), float("nan"), dtype=torch.float32, device=DEV)
    xb.xconv_pixel_dw_estimate(d, xb.to_device(dY, "f16", DEV), torch.from_numpy(xbar).to(DEV), dW,
                               xb.alloc_bytes(xb.xconv_pixel_workspace_bytes(d, xb.XCONV_OP_ESTIMATE), DEV))
    torch.cuda.synchronize()
    got = dW.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got)) and np.max(np.abs(got - want)) <= 2e-2 * np.max(np.abs(want))


# an infinity stays with its pixel and its channel's entries of Z: +-inf there, in the last channel (which the lanes of channels past the
# end read again) and in a middle one; every other pixel as without it
@pytest.mark.parametrize("hw", [(7, 7), (8, 8), (3, 37)])
@pytest.mark.parametrize("dtype,probe,C,r,nhwc", [("f32", "gaussian", 24, 12, False), ("f32", "rademacher", 33, 40, False), ("f32", "gaussian", 20, 64, True),
                                                  ("bf16", "rademacher", 40, 16, False), ("f16", "rademacher", 1, 36, False),
                                                  ("f16", "rademacher", 65, 64, False), ("bf16", "rademacher", 40, 24, True),
                                                  ("f16", "gaussian", 33, 12, False), ("bf16", "gaussian", 17, 64, False)])
def test_infinities(hw, dtype, probe, C, r, nhwc):
    if dtype != "f32" and probe == "gaussian" and hw[0] * hw[1] % 4 == 0:
        pytest.skip("aligned 16-bit planes take such a Z as a sum of two values, which an infinity times their opposite signs is not")
    (H, W), B = hw, 3
    X = synth.draw((B, C, H, W), 81, "normal", 1.0, dtype)
    dist, dt = (xo.GAUSSIAN if probe == "gaussian" else xo.RADEMACHER), {"f32": xo.F32, "bf16": xo.BF16, "f16": xo.F16}[dtype]
    Z = np.asarray(xo.probe_matrix(dist, 77, C, r)).reshape(C, r)
    want = xo.probe_fwd(X, Z, dt).copy()
    for b, c, y, x, v in [(0, C - 1, 0, 0, np.inf), (1, C // 2, H - 1, W - 1, -np.inf), (2, C - 1, H - 1, 1, -np.inf)]:
        X[b, c, y, x] = v
        want[b, :, y, x] = v * Z[c]
    d = xb.make_desc(B, C, 8, H, W, 1, 1, 0, r, dtype, probe, 77, xb.XCONV_NHWC if nhwc else xb.XCONV_NCHW)
    Xt = xb.alloc_xt(d, DEV)
    out = torch.empty((B, r, H, W), dtype=torch.float32, device=DEV)
    Xd = xb.to_device(X.transpose(0, 2, 3, 1) if nhwc else X, dtype, DEV)
    xb.xconv_probe_fwd(d, Xd, Xt, None, xb.alloc_ws(d, xb.XCONV_OP_PROBE, DEV))
    xb.xconv_xt_unpack(d, Xt, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    inf = np.isinf(want)
    assert inf.any() and np.array_equal(got[inf], want[inf])
    assert np.all(np.abs(got[~inf] - want[~inf]) <= TOL[dtype] * np.max(np.abs(want[~inf])))
