"""The calls by which this library's speed is judged: sizes, inputs, one pass of each, and what it has to move.

Every case is one kind of call a program makes through `paper_2501_13986_amd.binding`:

  conv    the fused convolution on a neighbour graph (forward: inference, backward: forces and training, step: both,
          double: training on forces), edges already in CSR order
  md      the same on a neighbour list that arrives unsorted and new with every call: CSR preparation, then the
          convolution forward and backward through the permutation
  csr     the CSR preparation alone, the synchronous entry point
  tp      the batched product (a model that gathers and scatters by itself), per-sample weights, uvu
  uvw     the batched product with one shared dense weight set (fp32)
  uvw_ps  the batched product with a dense weight tile per sample

The expected values (`exact`) are formed in fp64 with plain torch from Clebsch-Gordan coefficients computed here.
"""
from __future__ import annotations

from functools import lru_cache
from math import factorial, log, pi, sqrt

import numpy as np
import torch

from paper_2501_13986_amd import binding as b

# irreps of x, y, z: the layouts of this repository's benchmark and tests
IRREPS = {
    "mace": ("128x0e+128x1o+128x2e", "1x0e+1x1o+1x2e+1x3o", "128x0e+128x1o+128x2e+128x3o"),
    "mul96": ("96x0e+96x1o", "1x0e+1x1o+1x2e", "96x0e+96x1o+96x2e"),
    "mul32": ("32x0e+32x1o+32x2e", "1x0e+1x1o+1x2e+1x3o", "32x0e+32x1o+32x2e+32x3o"),
    "tiny": ("4x0e+4x1o", "1x0e+1x1o", "4x0e+4x1o+4x1e+4x2e"),
    "many": ("+".join(f"32x{l}{p}" for l in range(4) for p in "eo"), "1x0e+1x1o+1x2e+1x3o",
             "+".join(f"32x{l}{p}" for l in range(4) for p in "eo")),
    "nequip": ("32x0e+32x1o+32x2e", "1x0e+1x1o+1x2e", "32x0e+32x1o+32x2e"),
    "uneven": ("32x0e+16x1o+16x2e", "1x0e+1x1o+1x2e", "16x0e+32x1o+16x2e"),
    "diffdock": ("48x0e+10x1o+10x1e+48x0o", "1x0e+1x1o+1x2e", "48x0e+10x1o+10x1e+48x0o"),
    "wide64": ("64x0e+64x1o", "1x0e+1x1o", "64x0e+64x1o"),
}


def listed():
    return [
        # one small molecule, one evaluation of energy and forces: what counts is latency and the number of launches
        {"name": "conv step, small molecule", "kind": "conv", "op": "step", "irreps": "mul32", "dtype": "f32", "nodes": 27, "degree": 9},
        # inference on a protein-sized graph
        {"name": "conv fwd, 5000 nodes", "kind": "conv", "op": "fwd", "irreps": "mace", "dtype": "f32", "nodes": 5000, "degree": 32},
        # the largest graph: the gradient pass, which dominates a training step
        {"name": "conv bwd, 20000 nodes", "kind": "conv", "op": "bwd", "irreps": "mace", "dtype": "f32", "nodes": 20000, "degree": 40},
        # double precision, as molecular dynamics and the reference comparisons run it
        {"name": "conv step f64, 2503 nodes", "kind": "conv", "op": "step", "irreps": "mace", "dtype": "f64", "nodes": 2503, "degree": 32},
        # a narrow model (32 channels) on a large graph
        {"name": "conv step 32 ch, 10007 nodes", "kind": "conv", "op": "step", "irreps": "mul32", "dtype": "f32", "nodes": 10007, "degree": 36},
        # training on forces needs the second-order pass
        {"name": "conv double, 2000 nodes", "kind": "conv", "op": "double", "irreps": "mace", "dtype": "f32", "nodes": 2000, "degree": 32},
        # molecular dynamics of a narrow model: the neighbour list is rebuilt with every call
        {"name": "md step 32 ch, 3001 nodes", "kind": "md", "op": "step", "irreps": "mul32", "dtype": "f32", "nodes": 3001, "degree": 32},
        # a new large graph (a data loader's next sample)
        {"name": "csr, 20000 nodes", "kind": "csr", "op": "csr", "irreps": "none", "dtype": "i64", "nodes": 20000, "degree": 40},
        # the batched product of a training step
        {"name": "tp step, 50000 rows", "kind": "tp", "op": "step", "irreps": "mace", "dtype": "f32", "rows": 50000},
        # second-order pass of a model with both parities of every degree (68 paths)
        {"name": "tp double 68 paths", "kind": "tp", "op": "double", "irreps": "many", "dtype": "f32", "rows": 20011},
        # dense shared weights: a linear mixing of channels inside the product, training step
        {"name": "uvw step, 100000 rows", "kind": "uvw", "op": "step", "irreps": "nequip", "dtype": "f32", "rows": 100000},
        # dense weights per edge (docking models), training step
        {"name": "uvw_ps step, 25000 rows", "kind": "uvw_ps", "op": "step", "irreps": "diffdock", "dtype": "f32", "rows": 25000},
    ]


def draw(rng):
    most = max(_seconds(c) for c in listed())
    while True:
        kind = rng.choice(["conv", "conv", "conv", "md", "csr", "tp", "tp", "uvw", "uvw_ps"])
        c = {"kind": kind, "dtype": rng.choice(["f32", "f32", "f64"])}
        if kind in ("conv", "md", "csr"):
            c["nodes"] = int(round(2 ** rng.uniform(log(27, 2), log(20000, 2))))
            c["degree"] = rng.randint(6, 9) if c["nodes"] < 120 else rng.randint(8, 48)
        else:
            c["rows"] = int(round(2 ** rng.uniform(log(17, 2), log(100000, 2))))
        if kind == "conv":
            c["op"], c["irreps"] = rng.choice(["fwd", "bwd", "step", "double"]), rng.choice(["mace", "mace", "mul32", "mul96", "tiny"])
        elif kind == "md":
            c["op"], c["irreps"] = "step", rng.choice(["mace", "mul32", "mul96"])
        elif kind == "csr":
            c["op"], c["irreps"], c["dtype"] = "csr", "none", "i64"
        elif kind == "tp":
            c["op"], c["irreps"] = rng.choice(["fwd", "bwd", "step", "double"]), rng.choice(["mace", "mul32", "mul96", "many"])
        elif kind == "uvw":
            c["op"], c["irreps"], c["dtype"] = rng.choice(["fwd", "bwd", "step"]), rng.choice(["nequip", "uneven"]), "f32"
        else:
            c["op"], c["irreps"] = rng.choice(["fwd", "bwd", "step", "double"]), rng.choice(["diffdock", "wide64"])
        if _seconds(c) <= most:
            return c


def _seconds(case):
    """A measure of a case's cost (only to keep the drawn ones below the largest listed one)."""
    w = work(case)
    return max(w["bytes"] / 4e12, w["flops"] / 4e13)


# ---- the product's description: segments, paths, coefficients ---------------------------------------------------------

def _segments(text):
    out, off = [], 0
    for t in text.split("+"):
        mul, ir = t.split("x")
        l, p = int(ir[:-1]), 1 if ir[-1] == "e" else -1
        out.append((int(mul), l, p, off))
        off += int(mul) * (2 * l + 1)
    return out, off


@lru_cache(None)
def _paths(irreps):
    """Every allowed (x segment, y segment, z segment), in weight order."""
    X, Y, Z = (_segments(t)[0] for t in IRREPS[irreps])
    return [(a, c, d) for a in X for c in Y for d in Z if abs(a[1] - c[1]) <= d[1] <= a[1] + c[1] and d[2] == a[2] * c[2]]


def _dims(irreps, kind):
    dx, dy, dz = (_segments(t)[1] for t in IRREPS[irreps])
    dense = kind in ("uvw", "uvw_ps")
    return dx, dy, dz, sum(a[0] * (d[0] if dense else 1) for a, _, d in _paths(irreps))


def _to_real(l):
    """Rows: real basis m = -l..l; columns: complex basis."""
    u = np.zeros((2 * l + 1, 2 * l + 1), complex)
    u[l, l] = 1
    for m in range(1, l + 1):
        u[l + m, l + m], u[l + m, l - m] = (-1) ** m / sqrt(2), 1 / sqrt(2)
        u[l - m, l - m], u[l - m, l + m] = 1j / sqrt(2), -1j * (-1) ** m / sqrt(2)
    return u


@lru_cache(None)
def _coefficients(l1, l2, l3):
    """Real coupling tensor [2l1+1, 2l2+1, 2l3+1], sum over (i, j) of C C = identity, first nonzero positive."""
    f = factorial
    cg = np.zeros((2 * l1 + 1, 2 * l2 + 1, 2 * l3 + 1))
    for m1 in range(-l1, l1 + 1):
        for m2 in range(-l2, l2 + 1):
            m3 = m1 + m2
            if abs(m3) > l3:
                continue
            pre = sqrt((2 * l3 + 1) * f(l3 + l1 - l2) * f(l3 - l1 + l2) * f(l1 + l2 - l3) / f(l1 + l2 + l3 + 1))
            pre *= sqrt(f(l3 + m3) * f(l3 - m3) * f(l1 - m1) * f(l1 + m1) * f(l2 - m2) * f(l2 + m2))
            s = 0.0
            for k in range(l1 + l2 - l3 + 1):
                d = (k, l1 + l2 - l3 - k, l1 - m1 - k, l2 + m2 - k, l3 - l2 + m1 + k, l3 - l1 - m2 + k)
                if min(d) >= 0:
                    s += (-1) ** k / np.prod([float(f(t)) for t in d])
            cg[m1 + l1, m2 + l2, m3 + l3] = pre * s
    c = np.einsum("ia,jb,kc,abc->ijk", _to_real(l1), _to_real(l2), _to_real(l3).conj(), cg)
    c = c.real if np.abs(c.real).max() > np.abs(c.imag).max() else c.imag
    c[np.abs(c) < 1e-12] = 0
    return c * (sqrt(2 * l3 + 1) / np.linalg.norm(c)) * np.sign(c.ravel()[np.nonzero(c.ravel())[0][0]])


@lru_cache(None)
def _nonzeros(irreps):
    return [int(np.count_nonzero(_coefficients(a[1], c[1], d[1]))) for a, c, d in _paths(irreps)]


# ---- inputs -----------------------------------------------------------------------------------------------------------

@lru_cache(None)
def _plan(irreps, kind, dtype):
    """A program makes its plan when the model is defined and keeps it."""
    return b.Plan(*IRREPS[irreps], mode=b.CGTP_UVW if kind in ("uvw", "uvw_ps") else b.CGTP_UVU, shared_weights=kind == "uvw",
                  dtype=b.CGTP_F64 if dtype == "f64" else b.CGTP_F32, device=0)


def _harmonics(v, lmax):
    """Real spherical harmonics of unit vectors, degrees 0..lmax (<= 3), m = -l..l, sum over m of Y^2 = 2l + 1."""
    x, y, z = v.unbind(1)
    s3, s15, a, c, d = sqrt(3.0), sqrt(15.0), sqrt(70.0) / 4, sqrt(105.0), sqrt(42.0) / 4
    q = [torch.ones_like(x), s3 * y, s3 * z, s3 * x,
         s15 * x * y, s15 * y * z, 0.5 * sqrt(5.0) * (3 * z * z - 1), s15 * x * z, 0.5 * s15 * (x * x - y * y),
         a * y * (3 * x * x - y * y), c * x * y * z, d * y * (5 * z * z - 1), 0.5 * sqrt(7.0) * z * (5 * z * z - 3),
         d * x * (5 * z * z - 1), 0.5 * c * z * (x * x - y * y), a * x * (x * x - 3 * y * y)]
    return torch.stack(q[: (lmax + 1) ** 2], 1)


def _graph(g, nodes, degree):
    """Points uniform in a periodic cube; the nodes * degree / 2 closest pairs (a cutoff near 1), both ways, in random
    order: (recv, send, unit vectors)."""
    side = (nodes * (4.0 * pi / 3.0) / degree) ** (1.0 / 3.0)
    reach = 1.15 ** 2 if nodes > 2048 else 3 * side * side      # wide enough to hold that many pairs
    pos = torch.rand((nodes, 3), generator=g, device="cuda", dtype=torch.float64) * side
    ends, far = [], []
    for at in range(0, nodes, 2048):
        d2 = torch.zeros((min(2048, nodes - at), nodes), device="cuda", dtype=torch.float64)
        for k in range(3):
            d = pos[None, :, k] - pos[at:at + 2048, None, k]
            d2 += (d - side * torch.round(d / side)) ** 2
        r, s = torch.nonzero(torch.triu(d2 < reach, at + 1), as_tuple=True)
        ends.append(torch.stack([r + at, s]))
        far.append(d2[r, s])
    ends, near = torch.cat(ends, 1), torch.argsort(torch.cat(far))[:nodes * degree // 2]
    edges = torch.cat([ends[:, near], ends.flip(0)[:, near]], 1)
    edges = edges[:, torch.randperm(edges.shape[1], generator=g, device="cuda")]
    d = pos[edges[1]] - pos[edges[0]]
    d = d - side * torch.round(d / side)
    return edges[0].contiguous(), edges[1].contiguous(), d / d.norm(dim=1, keepdim=True)


def _inputs(case, seed):
    """The inputs alone, made from the seed: graph, features, harmonics, weights, upstream gradients."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float64 if case["dtype"] == "f64" else torch.float32
    draw_ = lambda *shape: torch.randn(shape, generator=g, device="cuda", dtype=dt)  # noqa: E731
    kind, s = case["kind"], {}
    graph = kind in ("conv", "md", "csr")
    if graph:
        s["recv"], s["send"], unit = _graph(g, case["nodes"], case["degree"])
        if kind == "csr":
            return s
        if kind == "conv":   # the user's per-edge data are in the sorted order already
            order = torch.argsort(s["recv"] * case["nodes"] + s["send"])
            s["recv"], s["send"], unit = s["recv"][order], s["send"][order], unit[order]
        N, R = case["nodes"], s["recv"].shape[0]
    else:
        N = R = case["rows"]
        unit = torch.randn((R, 3), generator=g, device="cuda", dtype=torch.float64)
        unit = unit / unit.norm(dim=1, keepdim=True)
    dx, dy, dz, nw = _dims(case["irreps"], kind)
    op = case["op"]
    s["x"], s["y"] = draw_(N, dx), _harmonics(unit, int(sqrt(dy)) - 1).to(dt).contiguous()
    scale = 1.0 if kind not in ("uvw", "uvw_ps") else 1.0 / sqrt(_segments(IRREPS[case["irreps"]][0])[0][0][0])
    s["W"] = draw_(nw).mul_(scale) if kind == "uvw" else draw_(R, nw).mul_(scale)
    if op != "fwd":
        s["gz"] = draw_(N, dz)
    if op == "double":
        s["La"], s["Lb"], s["LC"] = draw_(N, dx), draw_(R, dy), draw_(R, nw)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    kind, op = case["kind"], case["op"]
    s["case"] = case
    if kind == "csr":
        return s
    s["plan"] = _plan(case["irreps"], kind, case["dtype"])
    like = torch.empty_like
    if kind == "conv":   # made once per graph and kept
        s["row_ptr"], s["col"], _, s["t_row_ptr"], s["t_perm"] = b.cgtp_csr_from_coo(s["recv"], s["send"], case["nodes"])
    if kind == "md":     # buffers of a simulation: outputs of the preparation and its scratch
        V, E = case["nodes"], s["recv"].shape[0]
        new = lambda n: torch.empty(n, dtype=torch.int64, device="cuda")  # noqa: E731
        s["csr"] = (new(V + 1), new(E), new(E), new(V + 1), new(E))
        s["scratch"] = torch.empty(b.cgtp_csr_workspace_bytes(E, V), dtype=torch.uint8, device="cuda")
    if op in ("fwd", "step"):
        dz = _dims(case["irreps"], kind)[2]
        s["z"] = torch.empty((s["x"].shape[0], dz), dtype=s["x"].dtype, device="cuda")
    if op in ("bwd", "step"):
        s["gx"], s["gy"], s["gW"] = like(s["x"]), like(s["y"]), like(s["W"])
    if op == "double":
        s["Lx"], s["Ly"], s["LW"], s["Lgz"] = like(s["x"]), like(s["y"]), like(s["W"]), like(s["gz"])
    return s


def run(s):
    kind, op = s["case"]["kind"], s["case"]["op"]
    if kind == "csr":
        return b.cgtp_csr_from_coo(s["recv"], s["send"], s["case"]["nodes"])
    p, out = s["plan"], ()
    if kind == "md":
        csr = b.cgtp_csr_from_coo_async(s["recv"], s["send"], s["case"]["nodes"], s["csr"], s["scratch"])
        row_ptr, col, perm, t_row_ptr, t_perm = csr
        z = b.conv_forward_perm(p, s["x"], s["y"], s["W"], s["z"], row_ptr, col, perm)
        g = b.conv_backward_perm(p, s["x"], s["y"], s["W"], s["gz"], s["gx"], s["gy"], s["gW"], row_ptr, col, t_row_ptr, t_perm, perm)
        return (z,) + tuple(g)
    if kind == "conv":
        graph = (s["row_ptr"], s["col"])
        back = graph + (s["t_row_ptr"], s["t_perm"])
        if op == "double":
            return b.conv_double_backward(p, s["x"], s["y"], s["W"], s["gz"], s["La"], s["Lb"], s["LC"],
                                          s["Lx"], s["Ly"], s["LW"], s["Lgz"], *back)
        if op in ("fwd", "step"):
            out += (b.conv_forward(p, s["x"], s["y"], s["W"], s["z"], *graph),)
        if op in ("bwd", "step"):
            out += tuple(b.conv_backward(p, s["x"], s["y"], s["W"], s["gz"], s["gx"], s["gy"], s["gW"], *back))
        return out
    if op == "double":
        return b.tp_double_backward(p, s["x"], s["y"], s["W"], s["gz"], s["La"], s["Lb"], s["LC"], s["Lx"], s["Ly"], s["LW"], s["Lgz"])
    if op in ("fwd", "step"):
        out += (b.tp_forward(p, s["x"], s["y"], s["W"], s["z"]),)
    if op in ("bwd", "step"):
        out += tuple(b.tp_backward(p, s["x"], s["y"], s["W"], s["gz"], s["gx"], s["gy"], s["gW"]))
    return out


# ---- what a pass cannot do without ------------------------------------------------------------------------------------

def work(case):
    kind, op = case["kind"], case["op"]
    graph = kind in ("conv", "md", "csr")
    V = case.get("nodes", 0)
    E = V * case["degree"] // 2 * 2 if graph else 0
    if kind == "csr":   # two index lists in; row_ptr, col, perm, t_row_ptr, t_perm out
        return {"bytes": 8 * (2 * E + 3 * E + 2 * (V + 1)), "flops": 0}
    el = 8 if case["dtype"] == "f64" else 4
    dx, dy, dz, nw = _dims(case["irreps"], kind)
    N, R = (V, E) if graph else (case["rows"], case["rows"])
    dense = kind in ("uvw", "uvw_ps")
    wrows = 1 if kind == "uvw" else R
    paths = _paths(case["irreps"])
    cg = sum(2 * n * a[0] for n, (a, _, _) in zip(_nonzeros(case["irreps"]), paths))
    wt = sum(2 * (2 * d[1] + 1) * a[0] * (d[0] if dense else 1) for a, _, d in paths)
    x, y, z, w = N * dx * el, R * dy * el, N * dz * el, wrows * nw * el
    index = (2 * R + V) * 8 if graph else 0   # row pointers and the other end of every edge, the transposed walk as well
    ops = ("fwd", "bwd") if op == "step" else (op,)
    total = {"bytes": 0, "flops": 0}
    for o in ops:
        if o == "fwd":
            moved, flops = x + y + w + z + index // 2, cg + wt
        elif o == "bwd":    # x, y, W, gz in; gx, gy, gW out
            moved, flops = 2 * (x + y + w) + z + index, 3 * cg + (2 * wt if dense else 3 * wt // 2)
        else:               # x, y, W, gz, La, Lb, LC in; Lx, Ly, LW, Lgz out
            moved, flops = 3 * (x + y + w) + 2 * z + index, (7 * cg + 5 * wt if dense else 8 * cg + 3 * wt)
        total["bytes"] += moved
        total["flops"] += R * flops
    if kind == "md":
        total["bytes"] += 8 * (2 * E + 3 * E + 2 * (V + 1))
    return total


def tolerance(case):
    if case["kind"] == "csr":
        return "exact"
    # about four times what these paths show against fp64 (2e-7 to 7e-7 in fp32, 1e-16 to 6e-16 in fp64; largest single
    # difference about 3e-6 and 6e-15 of the rms): sums in another order
    return {"rel": 4e-15, "max": 4e-14} if case["dtype"] == "f64" else {"rel": 3e-6, "max": 2e-5}


# ---- the same in fp64 with plain torch ----------------------------------------------------------------------------------

def _product(case, x, y, W):
    """z of every row, fp64."""
    kind, rows, off = case["kind"], x.shape[0], 0
    dz = _segments(IRREPS[case["irreps"]][2])[1]
    parts = {}
    for (mx, l1, _, ox), (_, l2, _, oy), (mz, l3, _, oz) in _paths(case["irreps"]):
        C = torch.from_numpy(_coefficients(l1, l2, l3)).to(x.device)
        A = (y[:, oy:oy + 2 * l2 + 1] @ C.permute(1, 0, 2).reshape(2 * l2 + 1, -1)).reshape(rows, 2 * l1 + 1, 2 * l3 + 1)
        t = x[:, ox:ox + mx * (2 * l1 + 1)].reshape(rows, mx, 2 * l1 + 1) @ A      # [rows, mul_x, 2 l3 + 1]
        if kind in ("uvw", "uvw_ps"):
            n = mx * mz
            w = W[off:off + n].reshape(mx, mz) if kind == "uvw" else W[:, off:off + n].reshape(rows, mx, mz)
            t = (t.transpose(1, 2).contiguous() @ w).transpose(1, 2)
        else:
            n = mx
            t = t * W[:, off:off + n, None]
        off += n
        t = t.reshape(rows, -1)
        parts[oz] = parts[oz] + t if oz in parts else t
    z, at = [], 0
    for oz in sorted(parts):
        if oz > at:
            z.append(x.new_zeros((rows, oz - at)))
        z.append(parts[oz])
        at = oz + parts[oz].shape[1]
    if at < dz:
        z.append(x.new_zeros((rows, dz - at)))
    return torch.cat(z, 1)


def exact(case, seed):
    kind, op = case["kind"], case["op"]
    if kind == "csr":   # whole numbers
        return None
    s = _inputs(case, seed)
    graph = kind in ("conv", "md")
    x, y, W = s["x"].double(), s["y"].double(), s["W"].double()
    R = y.shape[0]
    zero = torch.zeros_like
    z = x.new_zeros((x.shape[0], _dims(case["irreps"], kind)[2]))
    a, c, d = zero(x), zero(y), zero(W)
    gz = s["gz"].double() if op != "fwd" else None
    La, Lb, LC = (s[k].double() for k in ("La", "Lb", "LC")) if op == "double" else (None, None, None)
    step = 8192

    def add(to, rows, v):
        to.index_add_(0, rows, v) if graph else to[rows].add_(v)

    for at in range(0, R, step):
        e = slice(at, min(R, at + step))
        src = s["send"][e] if graph else e
        dst = s["recv"][e] if graph else e
        xe, ye, We = x[src].clone(), y[e].clone(), (W.clone() if kind == "uvw" else W[e].clone())
        if op == "fwd":
            add(z, dst, _product(case, xe, ye, We))
            continue
        ge = gz[dst].clone()
        for t in (xe, ye, We, ge):
            t.requires_grad_(True)
        ze = _product(case, xe, ye, We)
        ga, gc, gd = torch.autograd.grad(ze, (xe, ye, We), ge, create_graph=op == "double")
        if op == "double":
            L = (ga * La[src]).sum() + (gc * Lb[e]).sum() + (gd * LC[e]).sum()
            ga, gc, gd, gg = torch.autograd.grad(L, (xe, ye, We, ge))
            add(z, dst, gg)
        elif op == "step":
            add(z, dst, ze.detach())
        add(a, src, ga)
        c[e] = gc
        if kind == "uvw":
            d += gd
        else:
            d[e] = gd
    if op == "fwd":
        return (z,)
    if op == "double":
        return a, c, d, z
    return ((z,) if op == "step" else ()) + (a, c, d)
