"""The fp32 forward pass of training layers with a ReLU against FP64: the input transforms, edges of the
tiles, channel remainders; and autograd takes this pass (equal bits)."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("mode", ["direct", "pool2", "up2cat"])
@pytest.mark.parametrize("Cx,C2,cout,H,W", [(32, 16, 32, 10, 18), (24, 8, 40, 2, 34), (64, 32, 96, 34, 16),
                                            (16, 16, 64, 182, 186)])
def test_train_forward(mode, Cx, C2, cout, H, W):
    """An error of at most 4e-6 of the summed magnitudes (fp32 accumulation of <= 865 terms)."""
    from paper_2602_08642_amd import autograd as ag, ops
    g = torch.Generator().manual_seed(Cx + H)
    C2 = C2 if mode == "up2cat" else 0
    h, w = (2 * H, 2 * W) if mode == "pool2" else (H // 2, W // 2) if C2 else (H, W)
    x = torch.randn(2, h, w, Cx, generator=g)
    x2 = torch.randn(2, H, W, C2, generator=g) if C2 else None
    wt = torch.randn(cout, 3, 3, Cx + C2, generator=g) / math.sqrt(9 * (Cx + C2))
    b = torch.randn(cout, generator=g) * 0.1
    spec = dict(name="a", cin=Cx + C2, cout=cout, k=3, relu=True)
    layer = ag.LayerRef(spec, wt.to(DEV).requires_grad_(), b.to(DEV).requires_grad_(), torch.float32)
    xd, x2d = x.to(DEV), None if x2 is None else x2.to(DEV)
    y = ag.conv(xd, layer, mode, x2d).detach()
    assert torch.equal(y, ops.conv2d(xd, spec, layer.packed_train, b.to(DEV), mode, x2d, train=True))
    t = x.double()
    if mode == "pool2":
        t = (t[:, ::2, ::2] + t[:, ::2, 1::2] + t[:, 1::2, ::2] + t[:, 1::2, 1::2]) * 0.25
    elif C2:
        t = torch.cat([t.repeat_interleave(2, 1).repeat_interleave(2, 2), x2.double()], -1)
    conv = lambda a, k: torch.nn.functional.conv2d(a.permute(0, 3, 1, 2), k.permute(0, 3, 1, 2), padding=1).permute(0, 2, 3, 1)
    ref = (conv(t, wt.double()) + b.double()).clamp(min=0)
    mag = conv(t.abs(), wt.double().abs()) + b.double().abs()
    assert bool(((y.cpu().double() - ref).abs() <= 4e-6 * mag).all())
