"""The convolution of small graphs, one workgroup per row: rows cut at the windows of a piece (just below, at and above a
piece, over many windows, two of them meeting in one window), no edge, one edge.  And the walks over edge ranges on the small graphs that the other tests take through the row kernels."""
import numpy as np
import pytest

from oracle import conv as oconv
from oracle.irreps import TPSpec
from paper_2501_13986_amd import synth
from tests._util import assert_close, memo
from tests import test_gpu_conv as conv_tests
from tests.test_gpu_conv import SPECS, dev
from tests.test_gpu_conv_shapes import check

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SPECS.update({
    "mul8": ("8x0e+8x1o", "1x0e+1x1o", "8x0e+8x1o+8x1e"),
    "mul20": ("20x0e+7x4e+12x1o", "1x0e+1x2e", "20x0e+3x7o+12x1o"),      # unequal: lanes beyond a multiplicity; segments of no path
    "mul32": ("32x0e+32x1o", "1x0e+1x1o+1x2e", "32x0e+32x1o+32x2e"),
})
# degrees of the rows, receivers and senders alike: pieces are of 32 to 512 edges
DEGREES = {
    "around_a_piece": [0, 127, 128, 129, 0, 1, 256, 257, 3, 513, 0],
    "hubs": [5, 700, 2, 0, 300, 130, 131, 9, 540],
    "no_edge_but_one": [0, 0, 1, 0],
}


def graph(name, seed=7):
    deg = DEGREES[name]
    recv = np.repeat(np.arange(len(deg)), deg)
    rng = np.random.default_rng(seed)
    return rng.permutation(recv).astype(np.int64), rng.permutation(recv).astype(np.int64), len(deg)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name", list(DEGREES))
@pytest.mark.parametrize("spec_name", ["small", "odd_row", "mul8", "mul20", "mul32", "mul75", "mul96"])
def test_rows_of_every_length(spec_name, name, prec):
    from paper_2501_13986_amd import binding as b
    spec = TPSpec(*SPECS[spec_name])
    plan = b.Plan(*SPECS[spec_name], dtype=b.CGTP_F64 if prec == "f64" else b.CGTP_F32, device=0)
    recv, send, V = graph(name)
    E = recv.shape[0]
    print(f"spec={spec_name} graph={name} prec={prec} V={V} E={E}", flush=True)
    row_ptr, col, perm, t_row_ptr, t_perm = oconv.csr_from_coo(recv, send, V)
    npdt, tdt = (np.float64, torch.float64) if prec == "f64" else (np.float32, torch.float32)
    x, gz = (synth.normal(i, (V, d)).astype(npdt) for i, d in ((1, spec.dim_x), (4, spec.dim_z)))
    y, W = (synth.normal(i, (E, d)).astype(npdt) for i, d in ((2, spec.dim_y), (3, spec.n_w)))
    new = lambda *shape: torch.full(shape, float("nan"), dtype=tdt, device="cuda")
    g = [dev(a) for a in (row_ptr, col, t_row_ptr, t_perm)]
    rz = memo(oconv.forward, spec, x, y, W, row_ptr, col)
    rx, ry, rW = memo(oconv.backward, spec, x, y, W, gz, row_ptr, col)
    back = np.empty_like(perm)      # the edge data in another order, reached through the permutation
    back[perm] = np.arange(E)
    for p in (None, dev(perm)):
        for call in range(2):       # the second call finds the counters of the hubs as the first one left them
            z, gx, gy, gW = new(V, spec.dim_z), new(V, spec.dim_x), new(E, spec.dim_y), new(E, spec.n_w)
            ys, Ws = (dev(y), dev(W)) if p is None else (dev(y[back]), dev(W[back]))
            if p is None:
                b.conv_forward(plan, dev(x), ys, Ws, z, g[0], g[1])
                b.conv_backward(plan, dev(x), ys, Ws, dev(gz), gx, gy, gW, *g)
            else:
                b.conv_forward_perm(plan, dev(x), ys, Ws, z, g[0], g[1], p)
                b.conv_backward_perm(plan, dev(x), ys, Ws, dev(gz), gx, gy, gW, *g, p)
            torch.cuda.synchronize()
            assert_close(z.cpu().numpy(), rz, prec, "z")
            assert_close(gx.cpu().numpy(), rx, prec, "gx")
            assert_close(gy.cpu().numpy(), ry if p is None else ry[back], prec, "gy")
            assert_close(gW.cpu().numpy(), rW if p is None else rW[back], prec, "gW")


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name", ["typical", "few_long_rows", "many_empty", "empty_ends", "single_edge"])
@pytest.mark.parametrize("spec_name", ["small", "mul32", "mul96"])
def test_edge_ranges_of_small_graphs(spec_name, name, prec, monkeypatch):
    monkeypatch.setenv("CGTP_CONV_ROWS", "0")
    check(spec_name, name, prec)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name", ["typical", "few_long_rows", "many_empty", "hub"])
def test_edge_ranges_of_two_workers_a_wave_through_the_permutation(name, prec, monkeypatch):
    monkeypatch.setenv("CGTP_CONV_ROWS", "0")
    conv_tests.test_conv_on_unsorted_edge_data_through_the_edge_permutation("mul32", name, prec)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name", list(DEGREES))
@pytest.mark.parametrize("spec_name", ["small", "odd_row", "mul8", "mul20", "mul32", "mul75", "mul96"])
def test_second_order_pass_of_rows_of_every_length(spec_name, name, prec):
    from paper_2501_13986_amd import binding as b
    spec = TPSpec(*SPECS[spec_name])
    plan = b.Plan(*SPECS[spec_name], dtype=b.CGTP_F64 if prec == "f64" else b.CGTP_F32, device=0)
    recv, send, V = graph(name)
    E = recv.shape[0]
    print(f"spec={spec_name} graph={name} prec={prec} V={V} E={E}", flush=True)
    row_ptr, col, perm, t_row_ptr, t_perm = oconv.csr_from_coo(recv, send, V)
    npdt, tdt = (np.float64, torch.float64) if prec == "f64" else (np.float32, torch.float32)
    x, gz, La = (synth.normal(i, (V, d)).astype(npdt) for i, d in ((1, spec.dim_x), (4, spec.dim_z), (5, spec.dim_x)))
    y, W, Lb, LC = (synth.normal(i, (E, d)).astype(npdt) for i, d in ((2, spec.dim_y), (3, spec.n_w), (6, spec.dim_y), (7, spec.n_w)))
    new = lambda *shape: torch.full(shape, float("nan"), dtype=tdt, device="cuda")
    ref = memo(oconv.double_backward, spec, x, y, W, gz, La, Lb, LC, row_ptr, col)
    for call in range(2):       # the second call finds the counters of the hubs as the first one left them
        out = [new(V, spec.dim_x), new(E, spec.dim_y), new(E, spec.n_w), new(V, spec.dim_z)]
        b.conv_double_backward(plan, *(dev(a) for a in (x, y, W, gz, La, Lb, LC)), *out, *(dev(a) for a in (row_ptr, col, t_row_ptr, t_perm)))
        torch.cuda.synchronize()
        for got, want, what in zip(out, ref, ("Lx", "Ly", "LW", "Lgz")):
            assert_close(got.cpu().numpy(), want, prec, what)


@pytest.mark.parametrize("fill", [0, 1, 255])
@pytest.mark.parametrize("spec_name", ["mul8", "mul32"])
def test_counts_left_behind_are_none_of_the_next_call(spec_name, fill, monkeypatch):
    """The counters of finished pieces as calls that overlapped (which is not allowed) would leave them: later calls are right."""
    monkeypatch.setenv("CGTP_ROW_CNT_FILL", str(fill))
    test_rows_of_every_length(spec_name, "hubs", "f32")
    test_second_order_pass_of_rows_of_every_length(spec_name, "hubs", "f32")


# degrees of the ordinary rows, then of a few long ones.  Rows above 2 048 take their receivers from memory, above 768 the
# second-order kernel of fewer waves; 140 000 edges are more than 1 024 of the smallest windows; with 360 000 edges the weights
# exceed the Infinity Cache (non-temporal streams) and 17 000 rows come in four rounds of workgroups or more
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("spec_name,V,degree,hubs", [("small", 2100, 3, (600, 1500, 257)), ("mul32", 2100, 3, (600, 1500, 257)), ("mul32", 1000, 5, (1200,)),
                                                     ("mul8", 900, 40, (70000, 30000)), ("small", 900, 40, (70000, 200000)),
                                                     ("mul32", 17000, 20, (20000, 600)), ("mul96", 8000, 12, (20000, 600))])
def test_long_rows_in_every_kind_of_row_kernel(spec_name, V, degree, hubs, prec, monkeypatch):
    """Against the walks by edge ranges in fp64 (which the oracle checks on smaller graphs), on graphs too large for the oracle."""
    from paper_2501_13986_amd import binding as b
    f64 = b.CGTP_F64
    plan = b.Plan(*SPECS[spec_name], dtype=f64 if prec == "f64" else b.CGTP_F32, device=0)
    with monkeypatch.context() as m:
        m.setenv("CGTP_CONV_ROWS", "0")
        ranges = b.Plan(*SPECS[spec_name], dtype=f64, device=0)
    g = torch.Generator(device="cuda")
    g.manual_seed(V + degree)
    deg = torch.full((V,), degree, device="cuda", dtype=torch.int64)
    for k, d in enumerate(hubs):
        deg[(k * V) // len(hubs) + 5] = d
    recv = torch.repeat_interleave(torch.arange(V, device="cuda"), deg)
    E = recv.shape[0]
    order = lambda: torch.randperm(E, generator=g, device="cuda")
    recv, send = recv[order()], recv[order()]
    print(f"spec={spec_name} V={V} E={E} prec={prec} entry=conv_forward/conv_backward/conv_double_backward(_perm)", flush=True)
    row_ptr, col, perm, t_row_ptr, t_perm = b.cgtp_csr_from_coo(recv, send, V)
    dims = [plan.dim_x, plan.dim_y, plan.n_w, plan.dim_z, plan.dim_x, plan.dim_y, plan.n_w]
    ins = [torch.randn((V if k in (0, 3, 4) else E, d), generator=g, device="cuda") for k, d in enumerate(dims)]

    def run(p, dt, x, y, W, gz, La, Lb, LC):
        new = lambda *shape: torch.full(shape, float("nan"), dtype=dt, device="cuda")
        x, y, W, gz, La, Lb, LC = (t.to(dt) for t in (x, y, W, gz, La, Lb, LC))
        out = {"z": new(V, p.dim_z), "gx": torch.empty_like(x), "gy": torch.empty_like(y), "gW": torch.empty_like(W), "zp": new(V, p.dim_z),
               "gxp": torch.empty_like(x), "gyp": torch.empty_like(y), "gWp": torch.empty_like(W), "Lx": torch.empty_like(x),
               "Ly": torch.empty_like(y), "LW": torch.empty_like(W), "Lgz": new(V, p.dim_z)}
        for t in out.values():
            t.fill_(float("nan"))
        o = list(out.values())
        b.conv_forward(p, x, y, W, o[0], row_ptr, col)
        b.conv_backward(p, x, y, W, gz, *o[1:4], row_ptr, col, t_row_ptr, t_perm)
        b.conv_forward_perm(p, x, y, W, o[4], row_ptr, col, perm)
        b.conv_backward_perm(p, x, y, W, gz, *o[5:8], row_ptr, col, t_row_ptr, t_perm, perm)
        b.conv_double_backward(p, x, y, W, gz, La, Lb, LC, *o[8:], row_ptr, col, t_row_ptr, t_perm)
        torch.cuda.synchronize()
        return out

    kernels = [(b.K_CONV_FWD, "cgtp_conv_fwd"), (b.K_CONV_BWD, "cgtp_conv_bwd")]
    for k, name in kernels:
        assert plan.conv_kernel(k, V, E) == name + "_row" and ranges.conv_kernel(k, V, E) == name
    if prec == "f32":      # (fp64: not every plan has the registers)
        assert plan.conv_kernel(b.K_CONV_DBL_BWD, V, E) == "cgtp_conv_dbl_row"
    want = run(ranges, torch.float64, *ins)
    for call in range(2):       # the second call finds the counters as the first one left them
        got = run(plan, torch.float64 if prec == "f64" else torch.float32, *ins)
        for what, ref in want.items():
            assert bool(torch.isfinite(got[what]).all()), what
            # as oracle comparisons: relative to the value or the root mean square, whichever is larger; sums of n terms in
            # fp32 err by about 2^-24 sqrt(n) of their own size, 3e-5 for 200 000 edges, and only hub rows are so long
            err = ((got[what].double() - ref).abs() / ref.abs().clamp(min=float(ref.square().mean().sqrt()))).max()
            assert float(err) <= (1e-10 if prec == "f64" else 1e-4), (what, float(err))
