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


RULE = r'''
#include <cstdio>
#include <cstring>
#include "conv_split.hpp"
using namespace cgtp;
int main() {
  char op[8];
  long long few, f64, cpl, spw, many, res, nt, V, E, word;
  while (std::scanf("%7s %lld %lld %lld %lld %lld %lld %lld %lld %lld %lld", op, &few, &f64, &cpl, &spw, &many, &res, &nt, &V, &E, &word) == 11)
    std::printf("%d\n", !std::strcmp(op, "fwd") ? (int)forward_by_rows(V, E) : !std::strcmp(op, "dbl") ? (int)double_by_rows(V, E, nt, (int)spw)
                      : backward_by_rows({few != 0, f64 != 0, (int)cpl, (int)spw, many != 0, res, nt}, V, E, E * word));
}
'''
# few channels, fp64, channels per lane, workers per wave, more than 128 registers, workgroups resident (plain; non-temporal, for "dbl"
# of the second-order kernel), then bytes of an edge's weights
PLAN = {"mace": ((0, 0, 2, 1, 1, 256, 768), 8704), "mul96": ((0, 0, 2, 1, 0, 512, 1280), 2688), "mul32": ((0, 0, 1, 2, 0, 1024, 2048), 2176),
        "mul32_f64": ((0, 1, 1, 2, 1, 512, 1024), 4352), "tiny": ((1, 0, 1, 16, 0, 1024, 1024), 96), "mace_dbl": ((0, 0, 1, 1, 1, 512, 512), 8704),
        "mul96_dbl": ((0, 0, 1, 1, 1, 768, 768), 2688), "mul32_dbl": ((0, 0, 1, 2, 1, 1024, 1024), 2176)}
# measured on both sides of each line: 0 by ranges, 1 by rows, 2 by rows with non-temporal streams
MEASURED = [("fwd", "mace", 20000, 0.1, 1), ("fwd", "mace", 20000, 1, 0), ("fwd", "mace", 20000, 7, 1), ("fwd", "mul32_f64", 20000, 2, 0),
            ("fwd", "mul32_f64", 9000, 2, 1), ("dbl", "mace_dbl", 300, 0.5, 1), ("dbl", "mace_dbl", 20000, 1, 0), ("dbl", "mace_dbl", 20000, 0.1, 1),
            ("dbl", "mace_dbl", 9000, 3, 1), ("dbl", "mace_dbl", 7000, 1, 0), ("dbl", "mul96_dbl", 9000, 1, 1), ("dbl", "mul96_dbl", 20000, 1, 0),
            ("dbl", "mul96_dbl", 20000, 2, 1), ("dbl", "mul32_dbl", 12000, 1, 1), ("dbl", "mul32_dbl", 20000, 3, 0), ("dbl", "mul32_dbl", 20000, 4, 1),
            ("bwd", "mace", 300, 2, 1), ("bwd", "mace", 800, 2, 0),
            ("bwd", "mace", 20000, 0.1, 0), ("bwd", "mace", 20000, 2, 0), ("bwd", "mace", 20000, 40, 2), ("bwd", "mace", 2000, 32, 0),
            ("bwd", "mul96", 1500, 1, 1), ("bwd", "mul96", 9000, 4, 0), ("bwd", "mul96", 3300, 6, 1), ("bwd", "mul32", 5000, 1, 1),
            ("bwd", "mul32", 20000, 2, 0), ("bwd", "mul32", 3000, 18, 1), ("bwd", "mul32_f64", 800, 1, 1), ("bwd", "mul32_f64", 5000, 3, 0),
            ("bwd", "mul32_f64", 12000, 36, 2), ("bwd", "tiny", 20000, 0.5, 1), ("fwd", "mul96", 20000, 4, 0),
            ("dbl", "mace_dbl", 20000, 0.25, 0), ("bwd", "mul32", 9000, 7, 2)]


def test_rows_of_few_edges_go_by_ranges_where_those_are_faster(tmp_path):
    (tmp_path / "rule.cpp").write_text(RULE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(tmp_path / "rule.cpp"), "-o", str(tmp_path / "rule")], check=True)
    text = "\n".join(" ".join(map(str, (op, *PLAN[p][0], V, int(V * deg), PLAN[p][1]))) for op, p, V, deg, _ in MEASURED)
    got = subprocess.run([str(tmp_path / "rule")], input=text, capture_output=True, text=True, check=True).stdout.split()
    assert [int(g) for g in got] == [m[-1] for m in MEASURED]
