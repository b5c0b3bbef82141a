"""Backward of the gathering pyramid where its tiles, edges and splat box end: images smaller than a
kernel, ragged tiles, motion that leaves the box and the image, gradient rows that are not whole
16-byte pieces; against FP64 gradients of the oracle (tolerance as test_gpu_backward.py)."""
import ctypes as C

import pytest
import torch

import procgen
from oracle import filt as ofilt
from tests.test_gpu_backward import _seed, assert_grad_close

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("motion", [3.0, 60.0])
@pytest.mark.parametrize("cfg", [(2, 2, 2, 2, 5, 3, 3), (1, 4, 6, 2, 7, 3, 3), (1, 2, 4, 2, 5, 2, 5),
                                 (1, 1, 3, 1, 5, 3, 3), (2, 20, 72, 3, 5, 3, 3), (1, 18, 36, 2, 3, 3, 3),
                                 (1, 10, 66, 2, 5, 2, 5)])
def test_pyramid_backward_edges(cfg, motion):
    from paper_2602_08642_amd import _lib as L, ops
    N, H, W, levels, KD, KU, KT = cfg
    g = torch.Generator().manual_seed(_seed(cfg, motion))
    Ks = procgen.kernel_channels(levels, KD, KU, KT, True)
    Ls = [torch.randn(N, H >> l, W >> l, 4, generator=g) for l in range(levels)]
    z = [torch.randn(N, H >> l, W >> l, ops.round_kstride(Ks[l], torch.float32), generator=g) for l in range(levels)]
    prev, gout = torch.randn(N, H, W, 4, generator=g), torch.randn(N, H, W, 4, generator=g)
    for t in Ls + [prev, gout]:
        t[..., 3] = 0
    mv = (torch.rand(N, H, W, 2, generator=g) * 2 - 1) * motion
    d = [[t.to(DEV) for t in ts] for ts in (Ls, z, [prev, mv, gout])]
    # gradient rows of K + 1 floats (element stores) through the C entry point
    glog = [torch.full((N, H >> l, W >> l, Ks[l] + 1), 7.0, device=DEV) for l in range(levels)]
    gL = [torch.empty_like(t) for t in d[0]]
    gprev = torch.zeros_like(d[2][0])
    lib = L.load()
    nb = lib.aps_denoise_pyramid_bwd_workspace_size(N, H, W, levels, KD, KU, KT, 1)
    ws = torch.full((nb,), 255, dtype=torch.uint8, device=DEV)
    arr = lambda ts: (C.c_void_p * L.APS_MAX_LEVELS)(*[t.data_ptr() for t in ts])  # noqa: E731
    ints = lambda ts: (C.c_int * L.APS_MAX_LEVELS)(*[t.shape[-1] for t in ts])  # noqa: E731
    L.check(lib.aps_denoise_pyramid_bwd(arr(d[0]), arr(d[1]), L.APS_F32, ints(z), levels, KD, KU, KT, ops._p(d[2][0]),
                                        ops._p(d[2][1]), N, H, W, ops._p(d[2][2]), arr(glog), L.APS_F32, ints(glog),
                                        arr(gL), ops._p(gprev), ops._p(ws), nb, ops._stream()), "pyramid_bwd")
    L64, z64 = [[t.double().requires_grad_(True) for t in ts] for ts in (Ls, z)]
    p64 = prev.double().requires_grad_(True)
    out = ofilt.denoise_pyramid(L64, z64, KD, KU, KT, p64, mv.double())[0]
    (out * gout.double()).sum().backward()
    for l in range(levels):
        # a 1 x 1 level: every tap reads the same pixel, so the logit gradient is zero by cancellation
        # (w_k (<g, v> - <g, y>) with y = v) and only its rounding is left
        if H >> l > 1 or W >> l > 1:
            assert_grad_close(glog[l][..., :Ks[l]], z64[l].grad[..., :Ks[l]], 1e-4, f"dlogits[{l}]")
        assert torch.all(glog[l][..., Ks[l]:] == 0)
        assert_grad_close(gL[l][..., :3], L64[l].grad[..., :3], 1e-4, f"dL[{l}]")
    assert_grad_close(gprev[..., :3], p64.grad[..., :3], 1e-4, "dprev")
