"""aps_conv2d_bwd_data refuses gradient rows padded into another 16-channel (fp32 3x3) or 32-channel chunk
than the operator was packed for.  Host-side checks: no pointer is read."""
import pytest


@pytest.mark.parametrize("Cout,ldy,k,dtype", [(33, 52, 3, "APS_F32"), (40, 64, 3, "APS_F32"), (25, 36, 3, "APS_F32"),
                                              (25, 40, 3, "APS_BF16"), (25, 36, 1, "APS_F32")])
def test_other_chunk(Cout, ldy, k, dtype):
    from paper_2602_08642_amd import _lib as L
    lib = L.load()
    assert lib.aps_status_string(lib.aps_conv2d_bwd_data(16, None, ldy, 1, 8, 8, Cout, 16, k, 32, getattr(L, dtype), 16, None)) \
        == lib.aps_status_string(lib.aps_conv2d_bwd_data(16, None, Cout - 1, 1, 8, 8, Cout, 16, k, 32, getattr(L, dtype), 16, None))
