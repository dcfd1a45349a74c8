"""What the shared-weight uvw forward's generated code has to keep (no GPU needed)."""
import os
import subprocess
import sys

import pytest

from paper_2501_13986_amd import binding as b, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PLANS = {
    "nequip": (synth.NEQUIP_X, synth.NEQUIP_Y, synth.NEQUIP_Z),
    "scalars_only": ("16x0e", "1x0e+1x1o+1x2e", "16x0e+16x1o+16x2e"),
}


@pytest.mark.parametrize("name", list(PLANS))
def test_lanes_exchange_y_through_lds_behind_a_wave_barrier(name):
    """A lane reads words of lds_yd that other lanes of its wave stored: a barrier has to stand between the stores of a
    tile and its reads, and between its reads and the stores of the wave's next tile."""
    p = b.Plan(*PLANS[name], mode=b.CGTP_UVW, shared_weights=True, dtype=b.CGTP_F32, device=-1)
    loop = p.source(b.K_TP_FWD).split("for (i64 t_ = ", 1)[1].split("const int wvu", 1)[0]
    p.close()
    kinds = []
    for line in loop.splitlines():
        if "wave_barrier()" in line:
            kinds.append("barrier")
        elif "lds_yd[" in line:
            kinds.append("store")
        elif "= lds_yd + " in line:
            kinds.append("load")
    assert "store" in kinds and "load" in kinds
    turns = [k for i, k in enumerate(kinds) if i == 0 or k != kinds[i - 1]]
    assert turns == ["barrier", "store", "barrier", "load"], turns


# private memory with every path over the components of z'; with the scalars' paths over x it is 1 092, 1 088 and 700 bytes
@pytest.mark.parametrize("x,y,z,most", [
    ("16x0e+16x1o+16x2e+16x3o", "1x0e+1x1o+1x2e+1x3o", "16x0e+16x1o+16x2e+16x3o", 600),
    ("32x0e+32x1o+32x2e+32x3o", "1x0e+1x1o+1x2e+1x3o", "16x0e+16x1o+16x2e+16x3o", 648),
    ("16x0e+16x0o+16x1e+16x1o+16x2e+16x2o", "1x0e+1x1o+1x2e+1x3o", "16x0e+16x0o+16x1e+16x1o+16x2e+16x2o", 520),
    (synth.NEQUIP_X, synth.NEQUIP_Y, synth.NEQUIP_Z, 0),
])
def test_the_form_with_less_private_memory_is_kept(x, y, z, most):
    """In a process of its own: the figures are the installed compiler's, and one that has imported torch uses torch's."""
    code = ("from paper_2501_13986_amd import binding as b\n"
            f"p = b.Plan({x!r}, {y!r}, {z!r}, mode=b.CGTP_UVW, shared_weights=True, dtype=b.CGTP_F32, device=-2)\n"
            "print(p.kernel_info(b.K_TP_FWD)['scratch'], 'lds_yd' in p.source(b.K_TP_FWD))")
    scratch, uses_x = subprocess.run([sys.executable, "-c", code], cwd=ROOT, check=True, capture_output=True, text=True).stdout.split()
    assert int(scratch) <= most, scratch
    assert (uses_x == "True") == (most == 0)
