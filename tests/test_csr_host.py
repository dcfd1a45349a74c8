"""The bucket path of the CSR preparation on the host (tests/_csr_host.py): every record in its place, every access in
bounds, and no workgroup with more than fits its LDS however uneven the degrees are."""
import pytest

from tests import _csr_host


@pytest.fixture(scope="module")
def exe():
    return _csr_host.build()


CASES = [  # nodes, edges, receivers, senders; whether a bucket of either side has to be cut
    (27, 243, "uniform", "uniform", (False, False)),
    (1, 4096, "uniform", "uniform", (False, False)),        # one workgroup, one row
    (300, 4000, "hub", "one", (False, False)),              # one workgroup, a row long enough for the radix order
    (4096, 4097, "uniform", "uniform", (False, False)),
    (4097, 1, "uniform", "uniform", (False, False)),        # more nodes than one workgroup takes
    (50000, 4000, "hub", "uniform", (False, False)),
    (20000, 4096, "uniform", "one", (False, True)),         # the sample is the whole list
    (1, 4097, "uniform", "uniform", (True, True)),          # more edges than a bucket for each row could hold
    (3, 30000, "uniform", "tail", (True, True)),
    (3001, 20000, "uniform", "uniform", (False, False)),
    (5000, 20000, "sorted", "uniform", (False, False)),
    (2, 4500, "one", "uniform", (True, False)),
    (2, 4500, "one", "one", (True, True)),                  # equal edges: only their place in the list tells them apart
    (5000, 30000, "hub", "uniform", (True, False)),
    (777, 20000, "two", "hub", (True, True)),
    (5000, 30001, "pad", "pad", (True, True)),
    (2000, 90000, "tail", "tail", (True, True)),            # a cut bucket whose samples are ordered by counting
    (3000, 15000, "bad", "hub", (False, True)),             # out-of-range indices
    (4194304, 9000, "hub", "pad", (True, True)),            # 56-bit records
]


@pytest.mark.parametrize("V,E,receivers,senders,cut", CASES)
def test_bucket_path(exe, V, E, receivers, senders, cut):
    status, text, seen = _csr_host.run(exe, V, E, receivers, senders)
    assert status == 0, text
    assert seen["path"] < 2, text
    assert seen["largest"] <= 4096, text
    if seen["path"] == 1:
        assert tuple(n > seen["buckets"] for n in seen["pieces"]) == cut, text


def test_bucket_that_the_sample_misses(exe):
    """Two thirds of the edges in one row, at places the sample does not look at: sorted in memory, still right."""
    status, text, seen = _csr_host.run(exe, 3000, 20000, "missed", "missed")
    assert status == 0 and seen["largest"] > 4096, text


def test_workspace_of_a_larger_graph_serves_every_smaller_one():
    from paper_2501_13986_amd import binding as b
    edges = sorted({1, 2, 100, 4000, 4095, 4096, 4097, 4500, 5000, 8192, 8193, 20000, 65536, 96032, 160000, 262145, 600001, 800000,
                    1048577, 2000000, 2097152} | {int(1.37 ** k) for k in range(1, 46)})   # as long as no library sort takes part
    nodes = sorted({1, 2, 3, 50, 1000, 1024, 1025, 3001, 4095, 4096, 4097, 5000, 20000, 65536, 65537, 300000, 4194304} | {2 ** k + 1 for k in range(22)})
    size = {(E, V): b.cgtp_csr_workspace_bytes(E, V) for E in edges for V in nodes}
    assert min(size.values()) > 0
    for i, E in enumerate(edges):
        for j, V in enumerate(nodes):
            if i:
                assert size[edges[i - 1], V] <= size[E, V], (edges[i - 1], E, V)
            if j:
                assert size[E, nodes[j - 1]] <= size[E, V], (E, nodes[j - 1], V)
