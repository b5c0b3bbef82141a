"""bf16 3x3 convolutions, tiled kernel: output rows at strides and bases that allow 16-byte stores and
at ones that allow 8 bytes only, channel blocks with a remainder, ragged tiles; nothing beyond a
pixel's channels is written."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("pad,off", [(0, 0), (8, 8), (4, 0), (8, 4)])
@pytest.mark.parametrize("cin,cout,H,W", [(48, 32, 17, 19), (64, 48, 1, 5), (40, 80, 16, 16), (64, 96, 190, 203)])
def test_output_rows(cin, cout, H, W, pad, off):
    """Against FP64 on the same bf16 operands: half a bf16 unit of the result and 2e-6 of the summed
    magnitudes (fp32 accumulation of <= 577 terms)."""
    from paper_2602_08642_amd import _lib as L, ops
    g = torch.Generator().manual_seed(cin + H)
    x = torch.randn(2, H, W, cin, generator=g).bfloat16()
    w = (torch.randn(cout, 3, 3, cin, generator=g) / math.sqrt(9 * cin)).bfloat16().float()
    b = torch.randn(cout, generator=g) * 0.1
    net = ops.Net([dict(name="a", cin=cin, cout=cout, k=3, relu=True)], {"a": (w, b)}, torch.bfloat16, DEV)
    _, packed, bias = net.layer("a")
    ld, canary = cout + pad, 7.0
    y = torch.full((2 * H * W * ld + 2 * off,), canary, dtype=torch.bfloat16, device=DEV)
    xd = x.to(DEV)
    L.check(L.load().aps_conv2d_fwd(xd.data_ptr(), None, 2, H, W, cin, 0, 0, packed.data_ptr(), bias.data_ptr(),
                                    cout, 3, 1, ops._dt(torch.bfloat16), y.data_ptr() + 2 * off, ld,
                                    ops._dt(torch.bfloat16), ops._stream()), "conv2d")
    y = y.cpu()
    rows = y[off:off + 2 * H * W * ld].view(2, H, W, ld)
    got = rows[..., :cout].double()
    conv = lambda t, k: torch.nn.functional.conv2d(t.permute(0, 3, 1, 2), k.permute(0, 3, 1, 2), padding=1).permute(0, 2, 3, 1)
    ref = (conv(x.double(), w.double()) + b.double()).clamp(min=0)
    mag = conv(x.double().abs(), w.double().abs()) + b.double().abs()
    half = torch.ldexp(torch.tensor(2.0 ** -9, dtype=torch.double), torch.frexp(ref)[1])  # 2^-8 2^floor(log2 |ref|)
    assert bool(((got - ref).abs() <= half + 2e-6 * mag).all())
    assert bool((rows[..., cout:] == canary).all()) and bool((y[:off] == canary).all())
    assert bool((y[off + 2 * H * W * ld:] == canary).all())
