"""16-bit layers whose correlation takes fewer waves along the output channels than would fit (plan_corr's estimate): the
estimate against the oracle, with the chosen shape and with every other one."""
import numpy as np
import pytest
import torch

from oracle import xconv_oracle as xo
from paper_2106_06998_amd import binding as xb
from paper_2106_06998_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# B, C_in, C_out, H, W, k, stride, r; the widest shape has 2 waves (136 channels) or 4 (200, 264)
CASES = [
    (9, 24, 136, 33, 33, 1, 1, 12),
    (9, 16, 200, 28, 38, 1, 1, 4),
    (17, 24, 200, 25, 47, 3, 1, 4),
    (16, 24, 264, 19, 45, 3, 1, 4),
    (17, 24, 264, 38, 41, 5, 2, 16),
]
# ... with output rows so narrow that the widest shape is taken: waves that split their k-steps have none (8 columns and 4 waves) or
# unequal numbers of them
NARROW = [
    (9, 24, 200, 32, 9, 3, 1, 12),
    (9, 16, 200, 20, 21, 5, 2, 4),
    (22, 24, 264, 6, 4, 3, 1, 16),
]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", CASES + NARROW, ids=["c%d-%dx%d-k%d-s%d" % (c[2], c[3], c[4], c[5], c[6]) for c in CASES + NARROW])
def test_fewer_waves_along_the_channels(case, dtype, monkeypatch):
    B, C, Co, H, W, k, s, r = case
    p = k // 2
    Ho, Wo = xo.out_extent(H, k, s, p), xo.out_extent(W, k, s, p)
    X = synth.draw((B, C, H, W), 51, "relu_normal", 1.0, dtype)
    dY = synth.draw((B, Co, Ho, Wo), 52, "normal", 1e-2, dtype)
    d = xb.make_desc(B, C, Co, H, W, k, s, p, r, dtype, "rademacher", 53)
    want = xo.dw_estimate(dY, X, xo.probe_matrix(xo.RADEMACHER, 53, C, r), k, k, (s, s), (p, p), {"bf16": xo.BF16, "f16": xo.F16}[dtype])
    Xd, dYd = xb.to_device(X, dtype, DEV), xb.to_device(dY, dtype, DEV)
    Xt = xb.alloc_xt(d, DEV)
    xb.xconv_probe_fwd(d, Xd, Xt, None, xb.alloc_ws(d, xb.XCONV_OP_PROBE, DEV))
    widest = 4 if Co > 192 else 2
    bytes_, waves = [], []
    for force in (None, 1, 2, 4):
        if force and force > widest:
            continue
        if force:
            monkeypatch.setenv("XCONV_CORR_WM", str(force))
        waves.append(xb.xconv_plan_info(d, xb.XCONV_OP_ESTIMATE)["WM"])
        ws = xb.alloc_ws(d, xb.XCONV_OP_ESTIMATE, DEV)
        bytes_.append(ws.numel())
        dW = torch.full((Co, C, k, k), float("nan"), dtype=torch.float32, device=DEV)
        xb.xconv_dw_estimate(d, dYd, Xt, None, dW, ws)
        torch.cuda.synchronize()
        # fp32 sums of equal inputs (the stored probe output may differ in single last places)
        assert np.max(np.abs(dW.cpu().numpy() - want)) <= 1e-3 * np.max(np.abs(want))
    assert waves[1:] == [w for w in (1, 2, 4) if w <= widest]
    assert waves[0] == widest if case in NARROW else waves[0] < widest and bytes_[0] <= bytes_[-1]
