"""CSR preparation at the sizes where its path or its bucket layout changes, and on graphs whose buckets do not fit the
LDS of a workgroup: bit-exact against the oracle, with and without the transpose."""
import numpy as np
import pytest

from oracle import conv as oconv

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [  # V, E, receivers, senders
    (4096, 4096, "uniform", "uniform"),      # the largest graph of one workgroup
    (4096, 4097, "uniform", "uniform"),      # the smallest with buckets
    (4097, 4096, "uniform", "uniform"),      # more nodes than one workgroup takes: buckets
    (4097, 4097, "uniform", "uniform"),
    (1, 4096, "uniform", "uniform"),         # one row, the whole LDS
    (1, 4097, "uniform", "uniform"),         # one bucket of one row, cut
    (2, 9001, "uniform", "uniform"),
    (3001, 96033, "uniform", "uniform"),
    (1025, 600001, "uniform", "uniform"),
    (300000, 500000, "uniform", "uniform"),
    (5000, 100001, "hub", "uniform"),        # half of the edges in one receiver
    (5000, 100001, "uniform", "hub"),
    (5000, 70000, "hub", "hub"),
    (777, 60000, "few", "few"),              # three rows only, all others empty
    (20000, 800000, "sorted", "uniform"),
    (2, 4500, "one", "uniform"),             # a bucket of one row, cut into pieces
    (2, 4500, "one", "one"),                 # of equal edges
    (60000, 2600000, "tail", "sorted"),      # the largest tiles; pieces between neighbouring samples
    (20000, 900000, "tail", "tail"),         # padding: equal edges at the end of the list
    (3000, 60000, "missed", "missed"),       # a row that no sampled edge enters: sorted in memory
    (4194304, 9000, "hub", "tail"),          # the most nodes of the bucket path
    (1000, 2097152, "uniform", "hub"),       # the most edges that buckets of any number of rows take
    (1000, 2097153, "uniform", "hub"),       # one more on few rows: sorts, 32-bit keys
    (65536, 2621440, "tail", "uniform"),     # the most edges that the buckets take at all
    (2000, 2700001, "uniform", "uniform"),   # more: sorts
    (70001, 2700001, "uniform", "uniform"),  # 64-bit keys
    (4194305, 4000, "uniform", "uniform"),   # more nodes than the buckets hold: sorts, 64-bit keys
]


def nodes(rng, V, E, how):
    a = rng.integers(0, V, E)
    if how == "hub":
        a[rng.random(E) < 0.5] = V // 3
    elif how == "few":
        a = np.array([0, V // 2, V - 1])[rng.integers(0, 3, E)]
    elif how == "sorted":
        a.sort()
    elif how == "one":
        a[:] = V - 1
    elif how == "tail":
        a[E - E // 9:] = V - 1
    elif how == "missed":                            # the sample: four neighbours from each of 1 024 equal parts
        run = np.arange(1024, dtype=np.int64)
        lo, hi = run * E // 1024, (run + 1) * E // 1024
        first = lo + ((((run * 2654435761) % 2 ** 32) * ((hi - lo - 4) // 2 + 1)) >> 32)
        looked_at = np.zeros(E, bool)
        looked_at[(first[:, None] + np.arange(4)).ravel()] = True
        a[~looked_at & (np.arange(E) % 3 != 0)] = V // 2
    return a.astype(np.int64)


@pytest.mark.parametrize("V,E,recv_how,send_how", CASES)
def test_csr_paths_bit_exact(V, E, recv_how, send_how):
    from paper_2501_13986_amd import binding as b
    print(f"V={V} E={E} receivers={recv_how} senders={send_how}", flush=True)
    rng = np.random.default_rng(V + E)
    recv, send = nodes(rng, V, E, recv_how), nodes(rng, V, E, send_how)
    recv[-3:], send[-3:] = recv[:3], send[:3]            # equal edges keep their order
    ref = oconv.csr_from_coo(recv, send, V)
    dr, ds = torch.from_numpy(recv).cuda(), torch.from_numpy(send).cuda()
    for n, g, r in zip(("row_ptr", "col", "perm", "t_row_ptr", "t_perm"), b.cgtp_csr_from_coo(dr, ds, V), ref):
        assert np.array_equal(g.cpu().numpy(), r), n
    ws = torch.full((b.cgtp_csr_workspace_bytes(E, V),), 255, dtype=torch.uint8, device="cuda")
    flag = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    out = tuple(torch.full((n,), -5, dtype=torch.int64, device="cuda") for n in (V + 1, E, E, V + 1, E))
    b.cgtp_csr_from_coo_async(dr, ds, V, out, ws, flag, transpose=False)
    torch.cuda.synchronize()
    assert int(flag.item()) == 0
    for n, g, r in zip(("row_ptr", "col", "perm"), out, ref):
        assert np.array_equal(g.cpu().numpy(), r), n
    assert torch.all(out[3] == -5) and torch.all(out[4] == -5)


@pytest.mark.parametrize("V,E", [(50, 900), (900, 30000), (4194305, 4000)])
@pytest.mark.parametrize("value", [-1, "V", 2 ** 40])
def test_csr_flags_out_of_range_indices_as_edge_zero_zero(V, E, value):
    """In every path; such an edge is treated as (0, 0)."""
    from paper_2501_13986_amd import binding as b
    value = V if value == "V" else value
    print(f"V={V} E={E} index={value}", flush=True)
    rng = np.random.default_rng(E)
    recv, send = nodes(rng, V, E, "uniform"), nodes(rng, V, E, "uniform")
    recv[E // 2], send[E // 3] = value, value
    dr, ds = torch.from_numpy(recv).cuda(), torch.from_numpy(send).cuda()
    with pytest.raises(b.CgtpError):
        b.cgtp_csr_from_coo(dr, ds, V)
    ws = torch.empty(b.cgtp_csr_workspace_bytes(E, V), dtype=torch.uint8, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = tuple(torch.full((n,), -5, dtype=torch.int64, device="cuda") for n in (V + 1, E, E, V + 1, E))
    b.cgtp_csr_from_coo_async(dr, ds, V, out, ws, flag)
    torch.cuda.synchronize()
    assert int(flag.item()) == 1
    for e in (E // 2, E // 3):
        recv[e] = send[e] = 0
    for n, g, r in zip(("row_ptr", "col", "perm", "t_row_ptr", "t_perm"), out, oconv.csr_from_coo(recv, send, V)):
        assert np.array_equal(g.cpu().numpy(), r), n


def test_csr_workspace_grows_beyond_the_buckets():
    from paper_2501_13986_amd import binding as b
    edges = [4096, 100000, 2097152, 2097153, 2400000, 2621440, 2621441, 3000000, 8000001]
    nodes = [1, 1000, 4096, 4097, 20000, 65536, 65537, 4194304, 4194305, 6000000]
    size = [[b.cgtp_csr_workspace_bytes(E, V) for V in nodes] for E in edges]
    print(size)
    for i, row in enumerate(size):
        assert row == sorted(row), (edges[i], row)
    for j in range(len(nodes)):
        col = [row[j] for row in size]
        assert col == sorted(col), (nodes[j], col)
