"""The fp32 row sweep (16 -> 32, 32 -> 32, 32 -> 64 channels): equal bits to the tiled fp32 kernel, which an
output row stride other than the channel count selects, at the edges of bands and segments and of the rule that
chooses between them (1024 segments of 8 rows)."""
import pytest
import torch

from test_gpu_conv_split import DEV, _weights

pytestmark = pytest.mark.gpu
# units of 16 -> 32: 4, 1026, 1023, 1024, 1088, 2800
SIZES = [(1, 9, 33), (513, 1, 33), (341, 3, 65), (1, 8, 32737), (8, 135, 241), (1, 640, 1100)]


def _layer(cin, cout, N, H, W):
    from paper_2602_08642_amd import ops
    g = torch.Generator().manual_seed(cin + cout + H)
    w, b = _weights(g, cout, cin)
    sp = dict(name="a", cin=cin, cout=cout, k=3, relu=True)
    net = ops.Net([sp], {"a": (w, b)}, torch.float32, DEV)
    return ops, torch.randn(N, H, W, cin, generator=g).to(DEV), net.layer("a"), w, b


@pytest.mark.parametrize("N,H,W", SIZES)
@pytest.mark.parametrize("cin,cout", [(16, 32), (32, 32), (32, 64)])
def test_training_pass(cin, cout, N, H, W):
    ops, x, (s, pk, b), _, _ = _layer(cin, cout, N, H, W)
    swept = ops.conv2d(x, s, pk, b, train=True)
    tiled = ops.conv2d(x, s, pk, b, train=True, ldy=cout + 4)
    assert torch.equal(swept, tiled[..., :cout])
