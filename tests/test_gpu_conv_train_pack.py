"""The weights of fp32 training layers are packed once per refresh, into a buffer that stays: the forward
passes of training and of inference read the same one (edges of the output tiles, odd input counts)."""
import pytest
import torch

from test_gpu_conv_split import DEV, _ref, _weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout", [(16, 48), (24, 40), (32, 32), (96, 80), (64, 144), (40, 16)])
def test_one_packing(cin, cout):
    from paper_2602_08642_amd import autograd as ag, ops
    g = torch.Generator().manual_seed(cin + cout)
    w, b = _weights(g, cout, cin)
    x = torch.randn(1, 19, 35, cin, generator=g)
    spec = dict(name="a", cin=cin, cout=cout, k=3, relu=True)
    wd = w.to(DEV).requires_grad_()
    layer = ag.LayerRef(spec, wd, b.to(DEV).requires_grad_(), torch.float32)
    held = layer.packed_train
    for k in range(2):
        # 4e-6 of the magnitudes: fp32 sums of at most 865 terms
        r = _ref(x.double(), w.double(), b.double()).clamp(min=0)
        mag = _ref(x.double().abs(), w.double().abs(), b.double().abs())
        for y in (ag.conv(x.to(DEV), layer).detach(), ops.conv2d(x.to(DEV), spec, layer.packed, b.to(DEV))):
            assert bool(((y.cpu().double() - r).abs() <= 4e-6 * mag).all())
        w = w * -1.5
        with torch.no_grad():
            wd.copy_(w)
        layer.refresh()
        assert layer.packed_train is held and layer.packed is held
