"""bf16 weight and bias gradients (aps_conv2d_bwd_weight) against FP64 at the edges of the row
sweep: bands of 32 columns and of rows cut raggedly, channel tiles of 32 cut by 1 to 43 outputs
and 8 to 48 inputs, an input tile that spans both tensors of the concat, padded and unaligned
gradient rows, more bands than one block, the ReLU mask with NaN and negative entries."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"
# (mode, Cx, C2, Cout, ksize, ldy, mask)
LAYERS = [("direct", 32, 0, 32, 3, 32, True), ("direct", 16, 0, 16, 3, 16, True), ("direct", 16, 0, 1, 3, 8, False),
          ("direct", 64, 0, 96, 3, 96, True), ("pool2", 32, 0, 64, 3, 64, True), ("up2cat", 64, 32, 32, 3, 32, True),
          ("up2cat", 16, 24, 40, 3, 40, True), ("direct", 8, 0, 37, 3, 37, True), ("direct", 40, 0, 43, 1, 48, False),
          ("pool2", 48, 0, 25, 1, 25, False)]


@pytest.mark.parametrize("N,H,W", [(1, 2, 6), (2, 10, 34), (1, 70, 96), (3, 36, 64)])
@pytest.mark.parametrize("mode,Cx,C2,Cout,k,ldy,mask", LAYERS)
def test_wgrad_matches_fp64(mode, Cx, C2, Cout, k, ldy, mask, N, H, W):
    from paper_2602_08642_amd import _lib as L, ops
    g = torch.Generator().manual_seed(H * W + Cx + Cout)
    bf = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16)  # noqa: E731
    x = bf(N, 2 * H, 2 * W, Cx) if mode == "pool2" else bf(N, H // 2, W // 2, Cx) if mode == "up2cat" else bf(N, H, W, Cx)
    x2 = bf(N, H, W, C2) if C2 else None
    dy = bf(N, H, W, ldy)
    dy[..., Cout:] = float("nan")      # channels past Cout are ignored
    y = None
    if mask:
        y = torch.relu(bf(N, H, W, Cout))
        y[:, 0, 0] = float("nan")      # not > 0
        y[:, -1, -1] = -1.0
    d = lambda t: None if t is None else t.to(DEV)  # noqa: E731
    lib = L.load()
    nb = lib.aps_conv2d_bwd_weight_workspace_size(N, H, W, Cx, C2, Cout, k)
    ws = torch.full((nb,), 255, dtype=torch.uint8, device=DEV)
    dw = torch.full((Cout, k, k, Cx + C2), 7.0, device=DEV)
    db = torch.full((Cout,), 7.0, device=DEV)
    m = {"direct": L.APS_CONV_DIRECT, "pool2": L.APS_CONV_POOL2, "up2cat": L.APS_CONV_UP2_CAT}[mode]
    xs = [d(t) for t in (x, x2, dy, y)]
    args = [ops._p(xs[0]), ops._p(xs[1]), m, N, H, W, Cx, C2, ops._p(xs[2]), ops._p(xs[3]), ldy, Cout, k, L.APS_BF16]
    L.check(lib.aps_conv2d_bwd_weight(*args, ops._p(dw), ops._p(db), ops._p(ws), nb, ops._stream()), "wgrad")
    dw2 = torch.empty_like(dw)         # again, without the bias: the same bits
    L.check(lib.aps_conv2d_bwd_weight(*args, ops._p(dw2), C.c_void_p(None), ops._p(ws), nb, ops._stream()), "wgrad")
    assert torch.equal(dw, dw2)

    X = x.double()
    if mode == "pool2":                # rounded to bf16, as the input transform
        f = x.float()
        X = (((f[:, 0::2, 0::2] + f[:, 0::2, 1::2]) + (f[:, 1::2, 0::2] + f[:, 1::2, 1::2])) * 0.25).to(torch.bfloat16).double()
    elif mode == "up2cat":
        X = torch.cat([X.repeat_interleave(2, 1).repeat_interleave(2, 2), x2.double()], -1)
    G = dy[..., :Cout].double()
    if mask:
        G = torch.where(y > 0, G, torch.zeros_like(G))
    r = k // 2
    Xp = torch.nn.functional.pad(X, (0, 0, r, r, r, r))
    G2 = G.reshape(-1, Cout)
    for ky in range(k):
        for kx in range(k):
            P = Xp[:, ky:ky + H, kx:kx + W].reshape(-1, Cx + C2)
            ref, mag = G2.t() @ P, G2.abs().t() @ P.abs()
            # products of bf16 are exact; a float32 sum: 1e-5 of the magnitude
            assert bool(((dw[:, ky, kx].double().cpu() - ref).abs() <= 1e-5 * mag + 1e-30).all()), (ky, kx)
    assert bool(((db.double().cpu() - G2.sum(0)).abs() <= 1e-5 * G2.abs().sum(0) + 1e-30).all())
