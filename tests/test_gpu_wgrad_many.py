"""bf16 weight gradients of many small images, where a wave walks several bands: against FP64, in the
workspace that the query gives, which stays within a few rounds of blocks."""
import pytest

import test_gpu_wgrad as wgrad


@pytest.mark.gpu
@pytest.mark.parametrize("mode,Cx,C2,Cout,k,N,H,W", [
    ("direct", 8, 0, 8, 3, 8192, 4, 4), ("direct", 8, 0, 8, 3, 8193, 4, 4), ("direct", 64, 0, 96, 3, 1500, 6, 5),
    ("up2cat", 64, 32, 32, 3, 2800, 4, 4), ("pool2", 40, 0, 33, 1, 3000, 3, 34)])
def test_many_images(mode, Cx, C2, Cout, k, N, H, W):
    wgrad.test_wgrad_matches_fp64(mode, Cx, C2, Cout, k, Cout, k == 3, N, H, W)


@pytest.mark.parametrize("N,H,W", [(64, 256, 256), (4096, 16, 16), (100000, 8, 8)])
def test_workspace_is_bounded(N, H, W):
    """256 up + 128 skip -> 128 channels: four rounds of 512 blocks of 32 x 32 channels, 9 taps and the bias
    in float32; and the fp32 path's bias sums, 1024 pixels each at the least."""
    from paper_2602_08642_amd import _lib as L
    size = L.load().aps_conv2d_bwd_weight_workspace_size(N, H, W, 256, 128, 128, 3)
    assert size <= max(4 * 512 * 38 * 1024, 40 << 20) + N * H * W * 128 * 4 // 32 + 4096
