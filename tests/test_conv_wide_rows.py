"""Plans whose rows are too wide for a workgroup's LDS keep every call: the kernels that walk row by row are left out."""
import numpy as np
import pytest

from oracle import conv as oconv
from oracle.irreps import TPSpec
from paper_2501_13986_amd import binding as b, synth

# x of 10 624 and 6 400 words: four rows of them are more than 160 KiB in fp32 and in fp64
PLANS = {
    "segments_of_no_path": ("64x0e+" + "+".join(["64x7o"] * 11), "1x0e", "64x0e", b.CGTP_F32),
    "both_parities_f64": ("+".join(f"128x{l}{p}" for l in range(5) for p in "eo"), "1x0e", "128x0e", b.CGTP_F64),
    "segments_of_no_path_f64": ("64x0e+" + "+".join(["64x7o"] * 6), "1x0e", "64x0e", b.CGTP_F64),
}


@pytest.mark.parametrize("name", list(PLANS))
def test_plan_is_created(name):
    *irreps, dt = PLANS[name]
    p = b.Plan(*irreps, dtype=dt, device=-2)
    assert p.dim_x * (8 if dt == b.CGTP_F64 else 4) * 4 > 160 * 1024
    assert p.kernel_info(b.K_CONV_DBL_BWD)["vgprs"] > 0
    p.close()


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(PLANS))
def test_second_order_pass(name):
    torch = pytest.importorskip("torch")
    from tests._util import assert_close
    *irreps, dt = PLANS[name]
    prec, npdt, tdt = ("f64", np.float64, torch.float64) if dt == b.CGTP_F64 else ("f32", np.float32, torch.float32)
    spec = TPSpec(*irreps)
    plan = b.Plan(*irreps, dtype=dt, device=0)
    V, E = 9, 70
    print(f"plan={name} V={V} E={E} entry=conv_double_backward", flush=True)
    rng = np.random.default_rng(3)
    graph = oconv.csr_from_coo(rng.integers(0, V, E), rng.integers(0, V, E), V)
    row_ptr, col, _, t_row_ptr, t_perm = graph
    rows = [(1, V, spec.dim_x), (2, E, spec.dim_y), (3, E, spec.n_w), (4, V, spec.dim_z), (5, V, spec.dim_x), (6, E, spec.dim_y), (7, E, spec.n_w)]
    ins = [synth.normal(i, (n, d)).astype(npdt) for i, n, d in rows]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    outs = [torch.full(s, float("nan"), dtype=tdt, device="cuda") for s in ((V, spec.dim_x), (E, spec.dim_y), (E, spec.n_w), (V, spec.dim_z))]
    b.conv_double_backward(plan, *map(dev, ins), *outs, *map(dev, (row_ptr, col, t_row_ptr, t_perm)))
    torch.cuda.synchronize()
    for got, want, what in zip(outs, oconv.double_backward(spec, *ins, row_ptr, col), ("Lx", "Ly", "LW", "Lgz")):
        assert_close(got.cpu().numpy(), want, prec, what)


def test_ordinary_plans_have_the_row_kernels(tmp_path, monkeypatch):
    """One that does not compile is left out without an error; these plans have all of them."""
    monkeypatch.setenv("CGTP_CACHE_DIR", str(tmp_path))
    b.Plan("32x0e+32x1o", "1x0e+1x1o", "32x0e+32x1o", dtype=b.CGTP_F32, device=-2).close()
    names = [f.name.rsplit("_", 1)[0] for f in tmp_path.iterdir()]
    for kernel in ("cgtp_conv_fwd_row", "cgtp_conv_bwd_row", "cgtp_conv_dbl_row", "cgtp_conv_row_sums"):
        assert kernel in names, (kernel, names)
