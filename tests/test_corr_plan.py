"""The tile that 16-bit correlations take (plan_corr's estimate): layers where fewer waves along the output channels were measured to be
slower than the widest shape keep out of them, and layers that gain by half keep them.  Host only."""
import pytest

from paper_2106_06998_amd import binding as xb

# B, C_in, C_out, H, W, k, stride, r, op, waves measured as slow; microseconds with 1, 2 and 4 waves along the output channels.  With one
# wave along them four split the k-steps of a row, of which rows of 4 columns have one, rows of 8 two, and 20 or 14 columns no whole number
SLOW = [
    ((229, 16, 472, 4, 4, 3, 1, 48), "estimate", 1),      # 48.2  40.1  39.2
    ((22, 16, 440, 14, 14, 3, 1, 16), "estimate", 1),     # 34.8  29.3  29.4
    ((18, 128, 238, 102, 7, 3, 1, 16), "estimate", 1),    # 48.4  41.7  43.8
    ((115, 128, 208, 38, 4, 3, 1, 80), "estimate", 1),    # 83.3  73.0  76.6
    ((256, 64, 512, 7, 7, 5, 2, 16), "estimate", 1),      # 53.8  45.3  46.1
    ((12, 16, 472, 14, 14, 5, 1, 16), "exact", 1),        # 46.8  40.0  42.0
    ((62, 48, 232, 7, 20, 3, 1, 8), "exact", 1),          # 48.3  42.1  43.4
]
# ... and the waves of the shape that takes less than half of the widest's time
GAIN = [
    ((256, 256, 256, 28, 28, 3, 1, 16), "estimate", 1),   # 60.7  69.6  124
    ((256, 128, 256, 28, 28, 3, 1, 48), "estimate", 1),   # 133   165   284
    ((39, 219, 200, 144, 98, 1, 1, 4), "estimate", 1),    # 99    156   292
    ((53, 96, 232, 71, 71, 5, 1, 80), "estimate", 2),     # 976   828   1816
]


def waves(case, op, dtype):
    B, C_in, C_out, H, W, k, s, r = case
    d = xb.make_desc(B, C_in, C_out, H, W, k, s, k // 2, r, dtype, "rademacher", 3)
    plan = xb.xconv_plan_info(d, xb.XCONV_OP_ESTIMATE if op == "estimate" else xb.XCONV_OP_EXACT)
    assert plan["ws"] == 0
    return plan["WM"]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_narrow_rows_do_not_split_over_waves_that_idle(dtype):
    for case, op, slow in SLOW:
        assert waves(case, op, dtype) > slow, case


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_small_tiles_where_partial_tiles_or_strips_cost(dtype):
    for case, op, best in GAIN:
        assert waves(case, op, dtype) == best, case
