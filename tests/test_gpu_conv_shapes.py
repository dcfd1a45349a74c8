"""The convolution where its lane map and its row merge change form: multiplicities just above a wave (two passes,
or three / four channels per lane), rows split over very many edge ranges, row widths that end inside a vector."""
import numpy as np
import pytest

from oracle import conv as oconv
from tests._util import assert_close, memo
from tests.test_gpu_conv import GRAPHS, SPECS, build, dev
from tests.test_gpu_conv_dbl import incoming

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PAR = "{0}x0e+{0}x0o+{0}x1e+{0}x1o+{0}x2e+{0}x2o+{0}x3e+{0}x3o"
SPECS.update({
    "mul65": ("65x0e+65x1o", "1x0e+1x1o", "65x0e+65x1o"),         # odd: two passes of one channel per lane
    "mul75": ("75x0e+75x1o", "1x0e+1x1o", "75x0e+75x1o"),         # three channels per lane (fp32)
    "mul130": ("130x0e+130x1o", "1x0e+1x1o", "130x0e+130x1o"),    # even, above 128, no divisor up to four that fits: two passes of two
    "mul256": ("256x0e+256x1o", "1x0e+1x1o", "256x0e+256x1o"),    # four channels per lane (fp32), two passes of two (fp64)
    # 68 paths: the wide map, the narrow one and one channel per lane in one plan, by what each kernel's registers allow
    "par96": (PAR.format(96), "1x0e+1x1o+1x2e+1x3o", PAR.format(96)),
    "par192": (PAR.format(192), "1x0e+1x1o+1x2e+1x3o", PAR.format(192)),
    "odd_row": ("3x0e+3x1o", "1x0e+1x1o", "3x0e+3x1o+3x1e"),      # rows of 12 and 21 words
})
GRAPHS.update({"hub": (3, 30000, ()),                             # thousands of ranges in one row
               "small_typical": (12, 150, (0, 7))})


def check(spec_name, graph, prec, double=True):
    b, spec, plan, (x, y, W, gz), (row_ptr, col, perm, t_row_ptr, t_perm), (V, E) = build(spec_name, graph, prec, seed=130)
    print(f"spec={spec_name} graph={graph} prec={prec} V={V} E={E}", flush=True)
    npdt, tdt = (np.float64, torch.float64) if prec == "f64" else (np.float32, torch.float32)
    new = lambda *shape: torch.full(shape, float("nan"), dtype=tdt, device="cuda")
    g = [dev(a) for a in (row_ptr, col, t_row_ptr, t_perm)]
    d = [dev(a) for a in (x, y, W)]
    z, out = new(V, spec.dim_z), [new(V, spec.dim_x), new(E, spec.dim_y), new(E, spec.n_w)]
    b.conv_forward(plan, *d, z, g[0], g[1])
    b.conv_backward(plan, *d, dev(gz), *out, *g)
    torch.cuda.synchronize()
    assert_close(z.cpu().numpy(), memo(oconv.forward, spec, x, y, W, row_ptr, col), prec, "z")
    for got, ref, what in zip(out, memo(oconv.backward, spec, x, y, W, gz, row_ptr, col), ("gx", "gy", "gW")):
        assert_close(got.cpu().numpy(), ref, prec, what)
    if not double:
        return
    La, Lb, LC = incoming(spec, V, E, npdt, 130)
    out = [new(V, spec.dim_x), new(E, spec.dim_y), new(E, spec.n_w), new(V, spec.dim_z)]
    b.conv_double_backward(plan, *d, dev(gz), dev(La), dev(Lb), dev(LC), *out, *g)
    torch.cuda.synchronize()
    for got, ref, what in zip(out, memo(oconv.double_backward, spec, x, y, W, gz, La, Lb, LC, row_ptr, col), ("Lx", "Ly", "LW", "Lgz")):
        assert_close(got.cpu().numpy(), ref, prec, what)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("spec_name", ["mul65", "mul75", "mul96", "mul130", "mul192", "mul256"])
def test_lane_maps_above_one_wave(spec_name, prec):
    check(spec_name, "empty_ends", prec)


@pytest.mark.parametrize("rows", ["0", "1"])      # 1: the same rows in windows of the row kernels
@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("spec_name", ["odd_row", "mul1", "small"])
def test_rows_split_over_thousands_of_ranges(spec_name, prec, rows, monkeypatch):
    monkeypatch.setenv("CGTP_CONV_ROWS", rows)
    check(spec_name, "hub", prec, double=spec_name == "odd_row")


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("spec_name", ["par96", "par192"])
def test_lane_maps_of_many_paths(spec_name, prec):
    check(spec_name, "small_typical", prec)
