"""fp32 3x3 convolutions on fp16 halves (conv_f32.hip) against FP64: magnitudes far from 1, tiles of
very different magnitudes, weights of tiny and zero channels, infinities, NaN and overflow, a concat
chunk that spans both tensors, padded gradient rows, and input rows beyond 32-bit byte offsets."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _conv(x, w, b, relu=False, mode="direct", x2=None):
    from paper_2602_08642_amd import ops
    sp = dict(name="a", cin=w.shape[3], cout=w.shape[0], k=3, relu=relu)
    net = ops.Net([sp], {"a": (w, b)}, torch.float32, DEV)
    s, pk, bb = net.layer("a")
    return ops.conv2d(x.to(DEV), s, pk, bb, mode, None if x2 is None else x2.to(DEV)).cpu()


def _ref(x, w, b):
    N, H, W, C = x.shape
    xp = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    out = b.expand(N * H * W, -1).clone()
    for ky in range(3):
        for kx in range(3):
            out = out + xp[:, ky:ky + H, kx:kx + W].reshape(-1, C) @ w[:, ky, kx].t()
    return out.view(N, H, W, -1)


def _weights(g, cout, cin):
    return torch.randn(cout, 3, 3, cin, generator=g) / math.sqrt(9 * cin), torch.randn(cout, generator=g) * 0.1


@pytest.mark.parametrize("scale", [1e-30, 1e-9, 1.0, 1e9, 1e30])
@pytest.mark.parametrize("cin,cout,H,W", [(16, 32, 9, 35), (40, 64, 24, 20), (64, 96, 190, 200)])
def test_magnitudes(cin, cout, H, W, scale):
    """Inputs at `scale`, the output channels' weights at scales of their own (one all zero): an error
    of at most 2e-6 of the magnitude (K <= 576 products, each to 2^-21, fp32 sums)."""
    g = torch.Generator().manual_seed(cin + H)
    x = torch.randn(1, H, W, cin, generator=g) * scale
    w, b = _weights(g, cout, cin)
    f = 10.0 ** torch.linspace(-6, 6, cout)
    f[3] = 0.0
    w, b = w * f.view(-1, 1, 1, 1), b * f * scale
    y = _conv(x, w, b).double()
    r = _ref(x.double(), w.double(), b.double())
    mag = _ref(x.double().abs(), w.double().abs(), b.double().abs())
    assert bool(((y - r).abs() <= 2e-6 * mag).all()), float(((y - r).abs() / (mag + 1e-300)).max())


def test_mixed_magnitudes():
    """One 16-row tile with parts 2^24 apart, and chunks whose largest element grows and shrinks: the
    error is also allowed 2^-49 of the tile's largest element per weight."""
    g = torch.Generator().manual_seed(5)
    x = torch.randn(1, 200, 208, 96, generator=g)
    x[:, 40:120] *= 2.0 ** -24
    x[..., :32] *= 2.0 ** -10
    x[..., 64:] *= 2.0 ** -5
    w, b = _weights(g, 64, 96)
    b = b * 0
    y = _conv(x, w, b).double()
    r = _ref(x.double(), w.double(), b.double())
    mag = _ref(x.double().abs(), w.double().abs(), b.double())
    floor = 2.0 ** -49 * float(x.abs().max()) * w.double().abs().sum((1, 2, 3))
    assert bool(((y - r).abs() <= 2e-6 * mag + floor).all())


@pytest.mark.parametrize("cin,cout", [(32, 32), (64, 128)])
def test_non_finite(cin, cout):
    """Infinities, NaN and products beyond the fp32 range come out as in an fp32 convolution, and the
    other outputs are those of the finite part."""
    g = torch.Generator().manual_seed(cin)
    x = torch.randn(2, 40, 50, cin, generator=g)
    w, b = _weights(g, cout, cin)
    clean = _conv(x, w, b)
    x[0, 5, 7, 3] = float("inf")
    x[0, 20, 30, 9] = float("-inf")
    x[0, 20, 31, 10] = float("inf")
    x[1, 10, 10, 0] = float("nan")
    x[1, 33, 49, 5] = 3.3e38          # rounds to infinity as a 16-bit float
    w[2, 1, 1, 5] = 4.0               # overflows fp32 with it
    y = _conv(x, w, b)
    r = _ref(x, w, b)                 # fp32
    assert torch.equal(torch.isnan(y), torch.isnan(r))
    assert torch.equal(torch.isposinf(y), torch.isposinf(r)) and torch.equal(torch.isneginf(y), torch.isneginf(r))
    assert bool(torch.isinf(y).any()) and bool(torch.isinf(y[1, 33, 49, 2]))
    touched = torch.nn.functional.max_pool2d((~(x.abs() < 1e30)).any(-1, keepdim=True).permute(0, 3, 1, 2).float(), 3, 1, 1)[:, 0] > 0
    ch = torch.arange(cout) != 2      # the channel whose weight was changed
    # fp32 rounding of sums below 10, also beside the outlier in the tile
    assert float((y - clean).abs()[~touched][:, ch].max()) <= 2e-6 * 10
    fin = touched.unsqueeze(-1) & torch.isfinite(r)
    assert bool(((y - r).abs()[fin] <= 1e-5 * r.abs()[fin] + 1e-4).all())
    relu = _conv(x, w, b, relu=True)  # NaN -> 0, as the rectifier of the other kernels
    assert not bool(torch.isnan(relu).any())


@pytest.mark.parametrize("Cx,C2,cout,H,W", [(16, 24, 32, 12, 20), (40, 64, 64, 10, 34)])
def test_concat_chunk_spans_both(Cx, C2, cout, H, W):
    g = torch.Generator().manual_seed(Cx + W)
    x = torch.randn(2, H // 2, W // 2, Cx, generator=g)
    x2 = torch.randn(2, H, W, C2, generator=g)
    w, b = _weights(g, cout, Cx + C2)
    y = _conv(x, w, b, mode="up2cat", x2=x2).double()
    X = torch.cat([x.repeat_interleave(2, 1).repeat_interleave(2, 2), x2], -1).double()
    r, mag = _ref(X, w.double(), b.double()), _ref(X.abs(), w.double().abs(), b.double().abs())
    assert bool(((y - r).abs() <= 2e-6 * mag).all())


def test_padded_gradient_rows():
    """aps_conv2d_bwd_data: channels of dy past Cout are ignored whatever they hold."""
    from paper_2602_08642_amd import _lib as L, ops
    g = torch.Generator().manual_seed(3)
    N, H, W, Cout, ldy, Cin = 1, 20, 24, 43, 44, 32
    w = torch.randn(Cout, 3, 3, Cin, generator=g) / 20
    dy = torch.randn(N, H, W, ldy, generator=g)
    dy[..., Cout:] = float("nan")
    pk = ops.pack_dgrad(dict(cin=Cin, cout=Cout, k=3), w.to(DEV), torch.float32)
    dX = torch.empty(N, H, W, Cin, device=DEV)
    d = dy.to(DEV)
    L.check(L.load().aps_conv2d_bwd_data(ops._p(d), None, ldy, N, H, W, Cout, ops._p(pk), 3, Cin, L.APS_F32,
                                         ops._p(dX), ops._stream()), "bwd_data")
    wt = w.flip(1, 2).permute(3, 1, 2, 0).double()
    G = dy[..., :Cout].double()
    r, mag = _ref(G, wt, torch.zeros(Cin).double()), _ref(G.abs(), wt.abs(), torch.zeros(Cin).double())
    assert bool(((dX.double().cpu() - r).abs() <= 2e-6 * mag).all())


def test_rows_beyond_32_bit_offsets():
    """An image whose 18 input rows are over 4 GiB: windows of it equal the convolution of the window."""
    from paper_2602_08642_amd import ops
    H, W, C = 18, 1900032, 32
    g = torch.Generator(device=DEV).manual_seed(1)
    x = torch.randn(1, H, W, C, generator=g, device=DEV)
    gw = torch.Generator().manual_seed(2)
    w, b = _weights(gw, 32, C)
    sp = dict(name="a", cin=C, cout=32, k=3, relu=False)
    net = ops.Net([sp], {"a": (w, b)}, torch.float32, DEV)
    s, pk, bb = net.layer("a")
    y = ops.conv2d(x, s, pk, bb)
    for x0 in (0, 950000, W - 64):
        win = x[:, :, max(x0 - 1, 0):x0 + 65].cpu().double()
        r = _ref(win, w.double(), b.double())[:, :, (1 if x0 else 0):][:, :, :64]
        got = y[:, :, x0:x0 + 64].cpu().double()
        assert got.shape == r.shape and float((got - r).abs().max()) <= 1e-5, x0
