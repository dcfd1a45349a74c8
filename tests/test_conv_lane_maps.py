"""The lane map of a convolution kernel follows from what the kernel compiles to (no GPU needed): plans with many paths
must not pay for channels per lane with private memory or with a wave per SIMD."""
import pytest

from paper_2501_13986_amd import binding as b

Y = "1x0e+1x1o+1x2e+1x3o"
WALKS = (b.K_CONV_FWD, b.K_CONV_BWD, b.K_CONV_DBL_FWD, b.K_CONV_DBL_BWD)


def both_parities(mul, lmax):
    return "+".join(f"{mul}x{l}{p}" for l in range(lmax + 1) for p in "eo")


# private memory of the second-order sender walk: with as many channels per lane as bring it to one pass it is 320, 1 332,
# 592, 732 and 1 912 bytes; the fp64 plan of degree 3 needs some with one channel per lane too
@pytest.mark.parametrize("mul,lmax,dtype,most", [(96, 3, b.CGTP_F32, 0), (192, 3, b.CGTP_F32, 0), (256, 2, b.CGTP_F32, 0),
                                                 (96, 2, b.CGTP_F64, 0), (96, 3, b.CGTP_F64, 804)])
def test_many_path_plans_stay_out_of_private_memory(mul, lmax, dtype, most):
    irr = both_parities(mul, lmax)
    p = b.Plan(irr, Y, irr, dtype=dtype, device=-2)
    info = {k: p.kernel_info(k) for k in WALKS}
    p.close()
    for k in WALKS:
        assert info[k]["scratch"] <= (most if k == b.K_CONV_DBL_BWD else 0), (k, info[k])
    if dtype == b.CGTP_F32:
        assert info[b.K_CONV_FWD]["vgprs"] <= 256 and info[b.K_CONV_DBL_FWD]["vgprs"] <= 256, info
