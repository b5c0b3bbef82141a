"""Weights of different magnitudes within an output channel in the fp32 3x3 convolutions on fp16 halves
(conv_f32.hip): zero weights stay zero, small ones keep their bits, and a channel whose weights are too far
apart for the halves (or not finite) is summed in plain fp32, equal to the training pass bit for bit."""
import math

import pytest
import torch

from test_gpu_conv_split import DEV, _conv, _ref, _weights

pytestmark = pytest.mark.gpu


def _check(x, w, b, y):
    """At most 2e-6 of the summed magnitudes: K <= 576 products, each to 2^-21, fp32 sums."""
    r = _ref(x.double(), w.double(), b.double())
    mag = _ref(x.double().abs(), w.double().abs(), b.double().abs())
    assert bool(((y.double() - r).abs() <= 2e-6 * mag).all()), float(((y.double() - r).abs() / (mag + 1e-300)).max())


@pytest.mark.parametrize("big", [1e5, 1e7])
@pytest.mark.parametrize("cin,cout", [(32, 32), (64, 64)])
def test_zero_weights_ignore_large_inputs(cin, cout, big):
    """Input channels that the layer ignores, at every position of a group of eight, hold values up to 1e7."""
    g = torch.Generator().manual_seed(cin)
    x = torch.randn(1, 24, 40, cin, generator=g)
    w, b = _weights(g, cout, cin)
    w[0] = 0.0
    w[0, 1, 1, 1] = 1.0            # a channel of one weight
    for co in range(1, cout):
        w[co, ..., co % 8::8] = 0.0
        x[..., co % 8::8] *= big if co == 4 else 1.0
    w[..., 4::8] = 0.0
    _check(x, w, b, _conv(x, w, b))


@pytest.mark.parametrize("s", [8, 16, 20, 24, 26, 27, 28, 36, 45, 60, 100])
@pytest.mark.parametrize("cin,cout", [(32, 32), (64, 64)])
def test_small_weights_keep_their_bits(cin, cout, s):
    """Half of a channel's weights at 2^-s of the others; the inputs of the large ones are zero, so the
    outputs are sums over the small ones only."""
    g = torch.Generator().manual_seed(cin + s)
    x = torch.randn(1, 20, 36, cin, generator=g)
    w, b = _weights(g, cout, cin)
    w[..., 1::2] *= 2.0 ** -s
    x[..., 0::2] = 0.0
    _check(x, w, b * 0, _conv(x, w, b * 0))


@pytest.mark.parametrize("mode", ["direct", "pool2", "up2cat"])
@pytest.mark.parametrize("Cx,C2,cout,H,W,odd", [(32, 16, 32, 10, 18, 3), (24, 8, 40, 2, 34, 39), (64, 32, 96, 34, 16, 70),
                                                (40, 24, 64, 182, 186, 5), (32, 32, 32, 190, 180, 31)])
def test_plain_channels(mode, Cx, C2, cout, H, W, odd):
    """One output channel with weights 2^70 apart: its block of channels equals the training pass bit for bit."""
    from paper_2602_08642_amd import autograd as ag, ops
    g = torch.Generator().manual_seed(Cx + H)
    C2 = C2 if mode == "up2cat" else 0
    h, w_ = (2 * H, 2 * W) if mode == "pool2" else (H // 2, W // 2) if C2 else (H, W)
    x = torch.randn(2, h, w_, Cx, generator=g).to(DEV)
    x2 = torch.randn(2, H, W, C2, generator=g).to(DEV) if C2 else None
    w, b = _weights(g, cout, Cx + C2)
    w[odd, 2, 0, 9] = 2.0 ** -70
    sp = dict(name="a", cin=Cx + C2, cout=cout, k=3, relu=True)
    net = ops.Net([sp], {"a": (w, b)}, torch.float32, DEV)
    s, pk, bb = net.layer("a")
    layer = ag.LayerRef(sp, w.to(DEV).requires_grad_(), b.to(DEV).requires_grad_(), torch.float32)
    y = ops.conv2d(x, s, pk, bb, mode, x2)
    t = ops.conv2d(x, s, layer.packed_train, bb, mode, x2, train=True)
    blk = 32 if cout <= 32 else 64
    lo = odd // blk * blk
    assert torch.equal(y[..., lo:lo + blk], t[..., lo:lo + blk])
    assert float((y - t).abs().max()) <= 1e-5 * float(t.abs().max())


def test_non_finite_weights():
    g = torch.Generator().manual_seed(1)
    x = torch.randn(1, 12, 20, 40, generator=g)
    w, b = _weights(g, 96, 40)
    w[3, 0, 2, 33] = float("inf")
    w[70, 1, 1, 0] = float("nan")
    y, r = _conv(x, w, b), _ref(x, w, b)
    assert torch.equal(torch.isnan(y), torch.isnan(r))
    assert torch.equal(torch.isposinf(y), torch.isposinf(r)) and torch.equal(torch.isneginf(y), torch.isneginf(r))
    fin = torch.isfinite(r)
    assert bool(fin.any()) and float((y - r).abs()[fin].max()) <= 1e-5 * float(r[fin].abs().max())


def test_data_gradient_of_spread_weights():
    """aps_conv2d_bwd_data with weights 2^-60 of the others, masked rows and padded ones."""
    from paper_2602_08642_amd import _lib as L, ops
    g = torch.Generator().manual_seed(2)
    N, H, W, Cout, Cin = 1, 20, 24, 44, 32
    w = torch.randn(Cout, 3, 3, Cin, generator=g) / 20
    w[1::2] *= 2.0 ** -60
    dy = torch.randn(N, H, W, Cout, generator=g)
    dy[..., 0::2] = 0.0
    ym = torch.randn(N, H, W, Cout, generator=g)
    pk = ops.pack_dgrad(dict(cin=Cin, cout=Cout, k=3), w.to(DEV), torch.float32)
    dX = torch.empty(N, H, W, Cin, device=DEV)
    d, m = dy.to(DEV), ym.to(DEV)
    L.check(L.load().aps_conv2d_bwd_data(ops._p(d), ops._p(m), Cout, N, H, W, Cout, ops._p(pk), 3, Cin, L.APS_F32,
                                         ops._p(dX), ops._stream()), "bwd_data")
    _check(dy * (ym > 0), w.flip(1, 2).permute(3, 1, 2, 0).contiguous(), torch.zeros(Cin), dX.cpu())
