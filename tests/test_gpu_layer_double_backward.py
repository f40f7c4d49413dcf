"""The bias gradient of a layer is linear in dY and can be differentiated again (create_graph=True), with either engine."""
import pytest
import torch

from paper_2106_06998_amd.layer import XConv2d
from test_gpu_conv import DEV, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("engine", ["library", "framework"])
@pytest.mark.parametrize("mode", ["channel", "multi", "independent"])
def test_bias_gradient_carries_a_graph(engine, mode):
    say("bias gradient with a graph: %s %s" % (engine, mode))
    torch.manual_seed(3)
    layer = XConv2d(8, 6, 3, r=4, padding=1, mode=mode, engine=engine, device=DEV)
    x = torch.randn(2, 8, 10, 12, device=DEV)
    dy = torch.randn(2, 6, 10, 12, device=DEV, requires_grad=True)
    v = torch.randn(6, device=DEV)
    db, = torch.autograd.grad(layer(x), [layer.bias], dy, create_graph=True)
    assert db.requires_grad
    # fp32 sums of 240 values against fp64 ones
    assert torch.allclose(db.double(), dy.double().sum((0, 2, 3)), rtol=0, atol=240 * 2.0 ** -24 * float(dy.detach().abs().sum((0, 2, 3)).max()))
    again, = torch.autograd.grad(db, [dy], v)
    assert torch.equal(again, v.view(1, -1, 1, 1).expand_as(dy))
    plain, = torch.autograd.grad(layer(x), [layer.bias], dy.detach())
    assert not plain.requires_grad
