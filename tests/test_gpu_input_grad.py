"""Transposes of the fused input transforms (aps_conv_input_grad): channel counts and bases that allow
16-byte accesses and ones that do not, rows shorter and longer than a workgroup, with and without
accumulation; equal to the same fp32 operations in the same order."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"
MODES = {"direct": 0, "pool2": 1, "up2cat": 2}


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("acc", [0, 1])
@pytest.mark.parametrize("Cx,C2,H,W,off", [(8, 16, 2, 2, 0), (5, 3, 4, 6, 0), (16, 8, 6, 10, 1),
                                           (32, 16, 4, 600, 0), (64, 32, 130, 34, 0)])
@pytest.mark.parametrize("mode", list(MODES))
def test_input_grad(mode, Cx, C2, H, W, off, acc, dt):
    from paper_2602_08642_amd import _lib as L, ops
    C2 = C2 if mode == "up2cat" else 0
    g = torch.Generator().manual_seed(Cx + H)
    new = lambda *s: torch.randn(*s, generator=g).to(dt)
    dX = new(2, H, W, Cx + C2)
    dx = new(2, 2 * H, 2 * W, Cx) if mode == "pool2" else new(2, H // 2, W // 2, Cx) if C2 else new(2, H, W, Cx)
    dx2 = new(2, H, W, C2) if C2 else None
    def dev(t):  # at `off` elements past an allocation's start
        if t is None:
            return None
        b = torch.zeros(t.numel() + off, dtype=dt, device=DEV)
        b[off:] = t.flatten().to(DEV)
        return b[off:]
    a, b, c = dev(dX), dev(dx), dev(dx2)
    L.check(L.load().aps_conv_input_grad(MODES[mode], a.data_ptr(), 2, H, W, Cx, C2, ops._dt(dt), b.data_ptr(), acc,
                                         c.data_ptr() if C2 else None, acc, ops._stream()), "input_grad")
    f = dX.float()
    if mode == "pool2":
        v = (0.25 * f).repeat_interleave(2, 1).repeat_interleave(2, 2)
    elif C2:
        q = f[..., :Cx]
        v = ((q[:, ::2, ::2] + q[:, ::2, 1::2]) + q[:, 1::2, ::2]) + q[:, 1::2, 1::2]
        assert torch.equal(c.cpu().view_as(dx2), (dx2.float() * acc + f[..., Cx:]).to(dt))
    else:
        v = f
    assert torch.equal(b.cpu().view_as(dx), (dx.float() * acc + v).to(dt))
