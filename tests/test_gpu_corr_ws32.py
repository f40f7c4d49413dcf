"""The fp32 correlation on fp32 matrix instructions with few workgroups: each walks through many steps, whole runs, strips and groups of
images.  (With the number of splits alone given, the kernel for split floats takes these layers.)"""
import pytest

from paper_2106_06998_amd import binding as xb
from test_gpu_parity import run_edge

pytestmark = pytest.mark.gpu

CASES = [
    ("runs", 11, 16, 16, 8, 8, 3, 1, 1, 8, "rademacher", "f32"),
    ("strips", 9, 48, 40, 7, 76, 3, 1, 1, 24, "gaussian", "f32"),
    ("stride2", 13, 32, 24, 11, 16, 3, 2, 1, 16, "rademacher", "f32"),
    ("five-rows", 6, 24, 70, 9, 12, 5, 1, 2, 12, "gaussian", "f32"),
]


@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("occ", ["1", "2"], ids=["one-wg-per-cu", "two-wg-per-cu"])
@pytest.mark.parametrize("e", CASES, ids=[e[0] for e in CASES])
def test_fp32_instructions_walk_across_image_groups(e, occ, splits, monkeypatch):
    monkeypatch.setenv("XCONV_WS32_SPLITS", str(splits))
    monkeypatch.setenv("XCONV_WS32_OCC", occ)
    name, B, C_in, C_out, H, W, k, stride, pad, r, probe, dtype = e
    d = xb.make_desc(B, C_in, C_out, H, W, k, stride, pad, r, dtype, probe, 13)
    for op in (xb.XCONV_OP_ESTIMATE, xb.XCONV_OP_EXACT):
        plan = xb.xconv_plan_info(d, op)
        assert plan["ws"] == 2 and plan["M_WG"] == 16 * plan["WM"] and plan["S"] == splits
    run_edge(e)
