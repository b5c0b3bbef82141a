"""Scatter over image sizes at the edges of its 32 x 32 tiles, one to five levels, even and odd widths
and bases that do not allow two pixels per load: equal to the same fp32 operations in the same order."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("mode", ["hard", "dasr"])
@pytest.mark.parametrize("H,W,levels,off", [(16, 16, 5, 0), (48, 80, 5, 0), (33, 47, 1, 0), (34, 66, 2, 1),
                                            (36, 100, 3, 0), (40, 72, 4, 0), (1, 1, 1, 0), (96, 32, 5, 1)])
def test_levels(H, W, levels, off, mode):
    from paper_2602_08642_amd import _lib as L, ops
    g = torch.Generator().manual_seed(H * W)
    s = torch.rand(2, H, W, generator=g) * 3.5 * (torch.rand(2, H, W, generator=g) < 0.6)
    extra = (torch.rand(2, H, W, generator=g) < 0.5).int()
    whole = s.floor().int()
    count = (s.round().int() if mode == "dasr" else whole + extra * (s > whole)).to(torch.uint8)
    flat = count.flatten().int()
    offset = (flat.cumsum(0) - flat).int()
    total = int(flat.sum())
    samples = torch.randn(total, 4, generator=g)
    n = max(0, total - 3)  # the last samples did not fit the caller's buffer
    ext = torch.cat([samples[:n], torch.zeros(8, 4)])
    acc = torch.zeros(2 * H * W, 3)
    for j in range(int(flat.max()) if total else 0):
        have = (flat > j) & (offset + j < n)
        acc = acc + torch.where(have[:, None], ext[(offset + j).clamp(max=n).long(), :3], torch.zeros(1))
    d = flat.float() if mode == "dasr" else s.flatten()
    want = [torch.where(d[:, None] > 0, acc / d[:, None], torch.zeros(1)).view(2, H, W, 3)]
    for _ in range(1, levels):
        p = want[-1]
        want.append(((p[:, ::2, ::2] + p[:, ::2, 1::2]) + (p[:, 1::2, ::2] + p[:, 1::2, 1::2])) * 0.25)

    def dev(t):
        b = torch.zeros(t.numel() + off, dtype=t.dtype, device=DEV)
        b[off:] = t.flatten().to(DEV)
        return b[off:]
    import ctypes as C
    out = [torch.full((2, H >> l, W >> l, 4), 9.0, device=DEV) for l in range(levels)]
    ptrs = (C.c_void_p * levels)(*[o.data_ptr() for o in out])
    ds, dc, do, dv = dev(s), dev(count), dev(offset), samples.to(DEV)
    L.check(L.load().aps_scatter_samples_ex(ds.data_ptr(), dc.data_ptr(), do.data_ptr(), dv.data_ptr() if n else None, n, 2,
                                            H, W, levels, ops._MODES[mode], 1.0, 1, 0, None, 0, ptrs,
                                            ops._stream()), "scatter")
    for o, w in zip(out, want):
        o = o.cpu()
        assert torch.equal(o[..., :3], w) and bool((o[..., 3] == 0).all())
