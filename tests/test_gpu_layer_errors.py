"""A layer that runs out of device memory raises torch.OutOfMemoryError, as torch's own layers do (batch-size finders and retry code
catch that type), and works again afterwards; other refusals stay plain RuntimeErrors."""
import pytest
import torch

from paper_2106_06998_amd.layer import SignReLU, XConv2d
from test_gpu_conv import DEV, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["forward", "backward", "relu"])
def test_out_of_memory_keeps_its_type(which):
    say("out of memory in %s" % which)
    layer = SignReLU() if which == "relu" else XConv2d(64, 64, 3, r=8, padding=1, device=DEV)
    x = torch.randn(16, 64, 128, 128, device=DEV, requires_grad=True)    # 64 MB, as are the output and its gradients
    dy = torch.randn(16, 64, 128, 128, device=DEV)
    y = layer(x) if which == "backward" else None
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (16 << 20)) / total)   # no room for 64 MB
    try:
        with pytest.raises(torch.OutOfMemoryError):
            torch.autograd.grad(y, [x], dy) if which == "backward" else layer(x)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    y = layer(x)
    dx, = torch.autograd.grad(y, [x], dy)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(y).all()) and bool(torch.isfinite(dx).all())


def test_refusals_stay_runtime_errors():
    layer = XConv2d(8, 4, 3, r=4, padding=1, device=DEV)
    with pytest.raises(RuntimeError, match="channels"):
        layer(torch.randn(2, 6, 8, 8, device=DEV))
    layer = XConv2d(8, 4, 3, r=2000, padding=1, device=DEV)
    with pytest.raises(RuntimeError, match="not supported"):
        layer(torch.randn(2, 8, 8, 8, device=DEV))
