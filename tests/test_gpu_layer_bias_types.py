"""A layer whose bias is not in the storage type of its input: the bias is added to the rounded product by the framework, and the
sum rounded once, as `y += bias` does."""
import pytest
import torch

from paper_2106_06998_amd.layer import XConv2d
from test_gpu_conv import DEV, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["channel", "multi", "independent"])
@pytest.mark.parametrize("dtype,bias_dtype", [(torch.bfloat16, torch.float32), (torch.float16, torch.float64), (torch.float32, torch.bfloat16)])
def test_bias_of_another_type(mode, dtype, bias_dtype):
    say("bias %s of a %s layer, %s" % (bias_dtype, dtype, mode))
    torch.manual_seed(3)
    m = XConv2d(16, 24, 3, r=4, padding=1, mode=mode, device=DEV, dtype=dtype)
    b = torch.randn(24, device=DEV, dtype=bias_dtype)
    m.bias = torch.nn.Parameter(b.clone())
    x = torch.randn(3, 16, 12, 8, device=DEV).to(dtype)
    y = m(x)
    m.bias = torch.nn.Parameter(torch.zeros(24, device=DEV, dtype=dtype))
    want = m(x).detach().clone()
    want += b.view(1, -1, 1, 1)
    assert y.dtype == dtype and torch.equal(y, want)


def test_refused_inputs():
    m = XConv2d(16, 24, 3, r=4, padding=1, device=DEV)
    for shape in [(2, 8, 9, 9), (2, 32, 9, 9), (16, 9, 9)]:
        with pytest.raises(RuntimeError):
            m(torch.zeros(shape, device=DEV))
