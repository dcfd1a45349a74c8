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
