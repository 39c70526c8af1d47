"""Whole-network inference where a workgroup's run of steps crosses columns
and images, starts in the middle of a column, or is a single step."""
import pytest
import torch

from paper_1703_02563_amd import learned as Lm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (40, 5, 1000),   # 2 steps a column, 3 steps a workgroup
    (1, 2600, 59),   # one column, 650 steps: runs start inside it
    (1, 4, 60), (1, 5, 61), (2, 3, 62), (1, 9, 64), (1, 8, 119),  # edges of a column and of a step
    (600, 1, 2),     # one step an image
])
@pytest.mark.parametrize("scale", [1.0, 1e-38])  # 1e-38: activations below the normal range
def test_runs_equal_the_layer_launches(shape, scale):
    net = Lm.DescNet(seed=5)
    g = torch.Generator().manual_seed(7)
    for k in range(3):
        net.b[k] = (torch.randn(net.b[k].shape, generator=g) * 0.1).cuda()
    if scale != 1.0:
        net.w[0] *= scale
        net.b[0] *= scale
        net.wb[0] = net.w[0].to(torch.bfloat16).view(torch.int16).reshape(net.wb[0].shape)
    x = net.input_from_images((torch.rand(shape, generator=g) * 255).round().to(torch.uint8).cuda())
    ref, got = net.forward(x), net.infer(x)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), ref.view(torch.int32))
