"""The convolution's workspace over the size of the graph (no GPU needed): what a call reserves must hold the pieces of every
form it can take, and must not fall with the number of edges, or a call on a smaller graph frees what a captured one uses."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2501_13986_amd", "csrc")

DRIVER = r'''
#include <cstdio>
#include "conv_split.hpp"
using namespace cgtp;
int main() {   // resident workers, workers per wave, workers of a row in the two row kernels, bytes of a row
  long long all, spw, w0, w1, row, E;
  while (std::scanf("%lld %lld %lld %lld %lld %lld", &all, &spw, &w0, &w1, &row, &E) == 6) {
    std::printf("%lld %lld", (long long)most_pieces(all, (int)spw, {w0, w1}, E, row), (long long)(2 * conv_ranges(all, (int)spw, E)));
    for (long long w : {w0, w1}) std::printf(" %lld", w ? (long long)(2 * row_windows(row_lg(w, E, row), E)) : 0LL);
    std::printf("\n");
  }
}
'''

# the fp32 and fp64 plans of 128 channels (forward, backward), of 32 and of 4 channels, a plan without row kernels, a row that the
# 32 MiB of pieces limit, and a machine with fewer resident workers than there may be windows
PLANS = [(2048, 1, 8, 8, 8192), (2048, 1, 8, 4, 4608), (1024, 1, 4, 4, 16384), (4096, 2, 8, 4, 2048), (65536, 16, 16, 16, 208),
         (2048, 1, 0, 0, 4608), (2048, 1, 8, 8, 20480), (512, 1, 8, 4, 4608), (768, 1, 1, 2, 160000)]


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("conv_split")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "driver.cpp"), "-o", str(d / "driver")], check=True)
    return str(d / "driver")


@pytest.mark.parametrize("plan", PLANS)
def test_reserved_pieces_hold_every_form_and_never_fall(exe, plan):
    edges = sorted({1, 2, 3, 100, 128000, 131072, 131073, 160000, 800000, 64000} | {int(1.13 ** k) for k in range(1, 190)} |
                   {(1024 << k) + d for k in range(20) for d in (-1, 0, 1)})
    text = "\n".join(" ".join(map(str, plan + (E,))) for E in edges)
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split("\n")[:-1]
    assert len(out) == len(edges)
    before, falls = 0, 0
    windows = most = 0
    for E, line in zip(edges, out):
        reserved, ranges, *rows = map(int, line.split())
        assert reserved >= max(ranges, *rows), (E, line)
        assert reserved >= before, (E, reserved, before)
        assert ranges >= most, (E, ranges, most)      # all that the two walks of the second-order pass reserve by
        most = ranges
        assert all(2 * r <= 2 * 2 * 1024 and r * plan[4] <= 32 << 20 for r in rows), (E, line)
        falls += rows[0] < windows
        before, windows = reserved, rows[0]
    assert falls > 0 or plan[2] == 0     # the windows themselves do fall
