"""Inputs of different magnitudes within a tile in the fp32 3x3 convolutions on fp16 halves (conv_f32.hip):
every element keeps its bits however large its neighbours are, an output depends on its own inputs only, and
equal inputs give equal bits whatever the image's size; the passes over one chunk and the plain products
that this takes, in every input transform and with the pooled output and the head."""
import math

import pytest
import torch

from test_gpu_conv_split import DEV, _conv, _ref, _weights
from test_gpu_conv_split_weights import _check

pytestmark = pytest.mark.gpu
SPREADS = [8, 20, 24, 25, 26, 27, 28, 30, 45, 60, 72, 75, 100, 120]


def _away(g, *shape):
    """Random signs, magnitudes in [2^-6, 1): a tile of them takes one pass."""
    return (torch.rand(shape, generator=g) * (1 - 2.0 ** -6) + 2.0 ** -6) * (torch.randint(0, 2, shape, generator=g) * 2 - 1)


@pytest.mark.parametrize("s", SPREADS)
@pytest.mark.parametrize("cin,cout,H", [(32, 32, 20), (96, 64, 20), (40, 32, 190)])
def test_small_inputs_keep_their_bits(cin, cout, H, s):
    """Half of the inputs at 2^-s of the others, whose weights are zero."""
    g = torch.Generator().manual_seed(cin + s)
    x = torch.randn(1, H, 4 * H // 3, cin, generator=g)
    x[..., 1::2] *= 2.0 ** -s
    w, b = _weights(g, cout, cin)
    w[..., 0::2] = 0.0
    _check(x, w, b * 0, _conv(x, w, b * 0))


def test_zero_weights_ignore_far_larger_inputs():
    """Inputs of 1e9 that the layer ignores, beside ones around 1."""
    g = torch.Generator().manual_seed(3)
    x = torch.randn(1, 24, 40, 64, generator=g)
    w, b = _weights(g, 64, 64)
    w[..., 4::8] = 0.0
    x[..., 4::8] *= 1e9
    _check(x, w, b, _conv(x, w, b))


@pytest.mark.parametrize("s", SPREADS)
@pytest.mark.parametrize("mode", ["direct", "pool2", "up2cat"])
def test_two_magnitudes(mode, s):
    """Inputs near 1 and near 2^-s in turn, the small ones with weights 2^s larger, so that both count."""
    from paper_2602_08642_amd import ops
    g = torch.Generator().manual_seed(s)
    Cx, C2, H, W, cout = 40, 24, 18, 34, 64
    C2 = C2 if mode == "up2cat" else 0
    h, w_ = (2 * H, 2 * W) if mode == "pool2" else (H // 2, W // 2) if C2 else (H, W)
    f = torch.where(torch.arange(Cx + C2) % 3 == 0, 1.0, 2.0 ** -min(s, 100))
    x = torch.randn(2, h, w_, Cx, generator=g) * f[:Cx]
    x2 = torch.randn(2, H, W, C2, generator=g) * f[Cx:] if C2 else None
    w, b = _weights(g, cout, Cx + C2)
    w = w / f
    t = x
    if mode == "pool2":
        t = ((x[:, ::2, ::2] + x[:, ::2, 1::2]) + (x[:, 1::2, ::2] + x[:, 1::2, 1::2])) * 0.25
    elif C2:
        t = torch.cat([x.repeat_interleave(2, 1).repeat_interleave(2, 2), x2], -1)
    _check(t, w, b, _conv(x, w, b, mode=mode, x2=x2))


def test_chunks_of_different_magnitudes():
    """Chunks whose scale rises and falls by up to 2^70, each with weights that bring it back to 1."""
    g = torch.Generator().manual_seed(9)
    f = torch.cat([torch.full((32,), 2.0 ** e) for e in (0, 35, -35, 30, -5)])
    x = torch.randn(1, 20, 40, 160, generator=g) * f
    w, b = _weights(g, 64, 160)
    _check(x, w, b, _conv(x, w, b))        # as they are: the large chunks decide
    w = w * 0
    w[..., 64:96] = _weights(g, 64, 32)[0]  # the smallest chunk alone
    _check(x, w, b * 0, _conv(x, w, b * 0))


@pytest.mark.parametrize("s", [30, 60, 90])
@pytest.mark.parametrize("cin,cout", [(32, 32), (64, 128)])
def test_outlier_leaves_its_neighbours_alone(cin, cout, s):
    """One element 2^s above the others: the outputs it does not reach have equal bits (s = 90, beyond what
    the passes cover: within the rounding of plain fp32 sums)."""
    g = torch.Generator().manual_seed(cin)
    x = _away(g, 1, 40, 50, cin)
    w, b = _weights(g, cout, cin)
    clean = _conv(x, w, b)
    x[0, 17, 21, 5] = 1.5 * 2.0 ** s
    y = _conv(x, w, b)
    far = torch.ones(40, 50, dtype=torch.bool)
    far[16:19, 20:23] = False
    if s <= 60:
        assert torch.equal(y[0, far], clean[0, far])
    _check(x, w, b, y)


@pytest.mark.parametrize("cin,cout", [(32, 32), (64, 64)])
def test_bits_do_not_depend_on_the_size(cin, cout):
    """A crop at odd offsets, alone (8-row tiles) and in a batch, equals the same pixels of the whole image."""
    g = torch.Generator().manual_seed(cin)
    x = _away(g, 1, 200, 190, cin) * 2.0 ** torch.randint(-18, 1, (1, 200, 190, cin), generator=g)
    w, b = _weights(g, cout, cin)
    y = _conv(x, w, b)
    crop = x[:, 33:75, 21:72]
    inner = y[:, 34:74, 22:71]
    assert torch.equal(_conv(crop, w, b)[:, 1:-1, 1:-1], inner)
    assert torch.equal(_conv(torch.cat([crop] * 20), w, b)[13:14, 1:-1, 1:-1], inner)


@pytest.mark.parametrize("kind", ["spread", "plain", "inf"])
@pytest.mark.parametrize("cin,cout", [(32, 32), (96, 64)])
def test_entry_points_agree(cin, cout, kind):
    """y of aps_conv2d_fwd, aps_conv2d_fwd_pool and aps_conv2d_fwd_head, bit for bit, where a tile takes several
    passes or plain products."""
    from paper_2602_08642_amd import _lib as L, ops
    g = torch.Generator().manual_seed(cin)
    N, H, W, K = 1, 34, 38, 43
    x = torch.randn(N, H, W, cin, generator=g)
    x[..., ::5] *= 2.0 ** -40
    if kind != "spread":
        x[0, 3, 5, 7] = float("inf") if kind == "inf" else 2.0 ** 100
    w, b = _weights(g, cout, cin)
    hw, hb = torch.randn(K, 1, 1, cout, generator=g) / math.sqrt(cout), torch.randn(K, generator=g)
    spec = [dict(name="a", cin=cin, cout=cout, k=3, relu=True), dict(name="h", cin=cout, cout=K, k=1, relu=False)]
    net = ops.Net(spec, {"a": (w, b), "h": (hw, hb)}, torch.float32, DEV)
    s, pk, bb = net.layer("a")
    _, hp, hbb = net.layer("h")
    xd = x.to(DEV)
    y = ops.conv2d(xd, s, pk, bb)
    y1, y2 = torch.empty_like(y), torch.empty_like(y)
    pool = torch.empty(N, H // 2, W // 2, cout, device=DEV)
    z = torch.empty(N, H, W, 44, device=DEV)
    L.check(L.load().aps_conv2d_fwd_pool(ops._p(xd), None, N, H, W, cin, 0, L.APS_CONV_DIRECT, ops._p(pk), ops._p(bb),
                                         cout, 1, L.APS_F32, ops._p(y1), ops._p(pool), ops._stream()), "pool")
    L.check(L.load().aps_conv2d_fwd_head(ops._p(xd), None, N, H, W, cin, 0, L.APS_CONV_DIRECT, ops._p(pk), ops._p(bb),
                                         cout, 1, ops._p(hp), ops._p(hbb), K, L.APS_F32, ops._p(y2), cout, ops._p(z),
                                         44, ops._stream()), "head")
    assert torch.equal(y, y1) and torch.equal(y, y2)
    mean = ((y[:, ::2, ::2] + y[:, ::2, 1::2]) + (y[:, 1::2, ::2] + y[:, 1::2, 1::2])) * 0.25
    assert torch.equal(pool, mean)
    ref = _ref(x, w, b).clamp(min=0)
    assert torch.equal(torch.isinf(y).cpu(), torch.isinf(ref)) if kind == "inf" else bool(torch.isfinite(y).all())
