"""aps_density_predict_bwd of an fp32 sampler wide enough for the fp16-halves convolutions: the signs that
its ReLU layers pass gradients by are those of the training forward pass, also for sums within rounding of
zero."""
import pytest
import torch

from test_gpu_conv_split import DEV, _weights

pytestmark = pytest.mark.gpu


def _conv64(x, w, b):
    return torch.nn.functional.conv2d(x.permute(0, 3, 1, 2), w.permute(0, 3, 1, 2), b, padding=1).permute(0, 2, 3, 1)


@pytest.mark.parametrize("C,c0,c1,H,W", [(32, 32, 32, 24, 40), (40, 64, 48, 18, 33)])
def test_gradient_signs(C, c0, c1, H, W):
    """Features constant over the image and first-layer biases that cancel the sums: away from the border every
    channel's sum is rounding noise.  The gradients, against FP64 with the training pass's signs, to
    1e-4 of their size (fp32 sums; one flipped channel changes its own by all of it)."""
    from paper_2602_08642_amd import ops
    g = torch.Generator().manual_seed(C)
    feat = torch.randn(C, generator=g).expand(1, H, W, C).contiguous().to(DEV)
    chans = [(C, c0), (c0, c1), (c1, 1)]
    spec = [dict(name="l%d" % i, cin=ci, cout=co, k=3, relu=i < 2) for i, (ci, co) in enumerate(chans)]
    wts = {s["name"]: list(_weights(g, s["cout"], s["cin"])) for s in spec}
    probe = ops.Net([dict(spec[0], relu=False)], {"l0": (wts["l0"][0], torch.zeros(c0))}, torch.float32, DEV)
    s, pk, b0 = probe.layer("l0")
    wts["l0"][1] = -ops.conv2d(feat, s, pk, b0, train=True)[0, H // 2, W // 2].cpu()
    net = ops.Net(spec, {k: tuple(v) for k, v in wts.items()}, torch.float32, DEV)
    a, h = [], feat
    for s in spec:
        _, pk, b = net.layer(s["name"])
        h = ops.conv2d(h, s, pk, b, train=True, ldy=4 if s["cout"] == 1 else None)
        a.append(h)
    split = ops.conv2d(feat, spec[0], *net.layer("l0")[1:])
    assert bool(((split > 0) != (a[0] > 0)).any())  # the two passes' signs do differ here
    gs = (torch.randn(1, H, W, generator=g) * 1e-2).to(DEV)
    grads, gfeat = ops.density_predict_bwd(net, feat, 0.25, gs)
    gz = ops.normalize_density_bwd(a[2][..., 0].contiguous(), 0.25, gs)
    x = feat.double().requires_grad_()
    p = [(net.master[s["name"]][0].double().requires_grad_(), net.master[s["name"]][1].double().requires_grad_()) for s in spec]
    h0 = _conv64(x, *p[0]) * (a[0] > 0)
    h1 = _conv64(h0, *p[1]) * (a[1] > 0)
    _conv64(h1, *p[2])[..., 0].backward(gz.double())
    pairs = [(gfeat, x.grad)] + [(q, r.grad) for s, pr in zip(spec, p) for q, r in zip(grads[s["name"]], pr)]
    for got, ref in pairs[:-1]:  # the last bias: its gradient is zero, as the normalisation ignores a shift
        d = (got.double() - ref).abs()
        assert bool((d <= 1e-4 * (ref.abs() + ref.square().mean().sqrt())).all()), float(d.max())
