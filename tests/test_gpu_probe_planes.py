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
