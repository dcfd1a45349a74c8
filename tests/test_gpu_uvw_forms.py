"""Shared-weight uvw plans whose products run over the components of x (paths from scalars to higher degrees), where the
form, its registers or its LDS change: multiplicities, batch sizes around the tiles, and plans that must keep the other form."""
import numpy as np
import pytest

from oracle import tp as otp
from oracle.irreps import Path, TPSpec, UVW
from paper_2501_13986_amd import synth
from tests._util import assert_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PLANS = {
    "scalars_only": ("16x0e", "1x0e+1x1o+1x2e", "16x0e+16x1o+16x2e"),
    "two_scalars": ("32x0e+16x0o", "1x1o+1x2e", "16x1o+32x2e+16x1e"),         # a y segment that starts after word 0, z reached twice
    "l3_coeff": ("16x0e+16x1o", "1x0e+1x3o", "32x3o+16x0e+16x2e", [(0, 1, 0, 1, -0.5), (0, 0, 1, 1, 2.0), (1, 1, 2, 1, 1.5)]),
    "nequip": (synth.NEQUIP_X, synth.NEQUIP_Y, synth.NEQUIP_Z),
    "degree3": ("16x0e+16x1o+16x2e+16x3o", "1x0e+1x1o+1x2e+1x3o", "16x0e+16x1o+16x2e+16x3o"),   # too many registers: z' form
    "wide_z": ("32x0e", "1x0e+1x1o+1x2e", "64x0e+64x1o+32x2e"),               # too many accumulators: z' form in the forward
}


@pytest.mark.parametrize("B", [1, 17, 1000, 40007])   # tiles of 16; whole tiles per wave from about 33 000 rows on
@pytest.mark.parametrize("name", list(PLANS))
def test_uvw_forms(name, B):
    from paper_2501_13986_amd import binding as b
    irr, paths = PLANS[name][:3], (PLANS[name][3] if len(PLANS[name]) > 3 else None)
    print(f"plan={name} B={B} entries=tp_forward/tp_backward uvw", flush=True)
    spec = TPSpec(*irr, paths=None if paths is None else [Path(*q) for q in paths], mode=UVW, shared_weights=True)
    plan = b.Plan(*irr, paths=paths, mode=b.CGTP_UVW, shared_weights=True, dtype=b.CGTP_F32, device=0)
    f = np.float32
    x, y = synth.normal(1, (B, spec.dim_x)).astype(f), synth.normal(2, (B, spec.dim_y)).astype(f)
    W, gz = synth.normal(3, spec.n_w, 0.2).astype(f), synth.normal(4, (B, spec.dim_z)).astype(f)
    dev = lambda a: torch.from_numpy(a).cuda()
    new = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda")
    z = b.tp_forward(plan, dev(x), dev(y), dev(W), new(B, spec.dim_z))
    g = b.tp_backward(plan, dev(x), dev(y), dev(W), dev(gz), new(B, spec.dim_x), new(B, spec.dim_y), new(spec.n_w))
    torch.cuda.synchronize()
    assert_close(z.cpu().numpy(), otp.forward(spec, x, y, W), "f32", "z")
    for got, ref, what in zip(g, otp.backward(spec, x, y, W, gz), ("gx", "gy", "gW")):
        assert_close(got.cpu().numpy(), ref, "f32", what)


@pytest.mark.parametrize("B", [1000, 40007])   # tiles split over a workgroup only; whole tiles and split ones
@pytest.mark.parametrize("name", list(PLANS))
def test_uvw_forward_row_does_not_depend_on_its_place(name, B):
    """Equal rows give equal results, bit for bit, whichever tile they are in."""
    from paper_2501_13986_amd import binding as b
    irr, paths = PLANS[name][:3], (PLANS[name][3] if len(PLANS[name]) > 3 else None)
    print(f"plan={name} B={B} entry=tp_forward uvw, equal rows", flush=True)
    plan = b.Plan(*irr, paths=paths, mode=b.CGTP_UVW, shared_weights=True, dtype=b.CGTP_F32, device=0)
    row = lambda seed, n: torch.from_numpy(synth.normal(seed, (1, n)).astype(np.float32)).cuda().expand(B, n).contiguous()
    W = torch.from_numpy(synth.normal(3, plan.n_w, 0.2).astype(np.float32)).cuda()
    z = b.tp_forward(plan, row(1, plan.dim_x), row(2, plan.dim_y), W, torch.full((B, plan.dim_z), float("nan"), device="cuda"))
    torch.cuda.synchronize()
    assert torch.equal(z, z[:1].expand(B, -1).contiguous())
