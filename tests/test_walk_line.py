"""The line between the walk with eight lanes per target and the 64-target walks
against measured times: per setting the largest measured number of targets at
which eight lanes were at least 1.2 times as fast (0: none that the line has to
reach), and the smallest at which they took more than 1 / 0.93 of the time
(host only: the rule is plain C++)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_17658_amd", "csrc")

# (walk, leaf_max, theta or alpha, particles of a list's box or 0: all targets, faster up to, slower from)
MEASURED = [
    ("mixed", 1, 0.1, 0, 16000, 80000), ("mixed", 2, 0.1, 0, 45000, 80000), ("mixed", 1, 0.2, 0, 16000, 45000),
    ("mixed", 2, 0.2, 0, 30000, 60000), ("mixed", 4, 0.2, 0, 45000, 110000), ("mixed", 8, 0.2, 0, 45000, 135000),
    ("mixed", 16, 0.2, 0, 60000, 160000), ("mixed", 1, 0.3, 0, 0, 110000), ("mixed", 2, 0.3, 0, 0, 110000),
    ("mixed", 4, 0.3, 0, 0, 160000), ("mixed", 1, 0.4, 0, 60000, 160000), ("mixed ext", 1, 0.2, 0, 0, 85000),
    ("mixed ext", 1, 0.2, 0, 0, 85000), ("mixed ext", 2, 0.2, 0, 30000, 110000),
    ("mixed ext", 2, 0.2, 0, 30000, 110000), ("mixed ext", 4, 0.2, 0, 60000, 160000),
    ("mixed ext", 1, 0.3, 0, 0, 160000), ("mixed ext", 1, 0.3, 0, 0, 160000),
    ("mixed relative", 1, 0.0005, 0, 85000, 135000), ("mixed relative", 1, 0.0001, 0, 60000, 110000),
    ("mixed relative", 2, 0.0001, 0, 85000, 135000), ("mixed", 1, 0.2, 300000, 75000, 110000),
    ("mixed", 4, 0.2, 300000, 75000, 150000), ("mixed", 1, 0.1, 700000, 60000, 100000),
    ("mixed", 1, 0.2, 700000, 60000, 100000), ("mixed", 1, 0.3, 700000, 0, 160000),
    ("mixed", 8, 0.3, 700000, 0, 175000), ("mixed", 1, 0.1, 3000000, 60000, 100000),
    ("mixed", 1, 0.2, 3000000, 100000, 160000), ("mixed", 2, 0.2, 3000000, 100000, 220000),
    ("mixed", 4, 0.2, 3000000, 0, 200000), ("mixed", 8, 0.2, 3000000, 100000, 220000),
    ("mixed", 1, 0.3, 3000000, 160000, 320000), ("mixed", 2, 0.3, 3000000, 160000, 320000),
    ("mixed", 4, 0.3, 3000000, 200000, 320000), ("mixed", 8, 0.3, 3000000, 160000, 320000),
    ("mixed newton", 1, 0, 0, 0, 25000), ("mixed newton", 1, 0.1, 0, 0, 3000),
    ("mixed newton", 1, 0.2, 0, 0, 55000), ("mixed newton", 4, 0.2, 0, 25000, 55000),
    ("mixed newton", 8, 0.2, 0, 25000, 55000), ("mixed newton", 1, 0.3, 0, 25000, 55000),
    ("mixed newton ext", 1, 0.2, 0, 25000, 70000), ("mixed newton", 1, 0.2, 1000000, 30000, 70000),
    ("mixed newton", 8, 0.2, 1000000, 30000, 100000), ("mixed newton", 1, 0.3, 1000000, 50000, 100000),
    ("mixed newton", 8, 0.3, 1000000, 50000, 100000), ("mixed newton", 1, 0.5, 1000000, 70000, 140000),
    ("mixed newton", 8, 0.5, 1000000, 70000, 140000), ("mixed newton", 8, 0.8, 1000000, 70000, 140000),
    ("fp64", 1, 0, 0, 30000, 150000), ("fp64", 1, 0.1, 0, 30000, 100000), ("fp64", 2, 0.1, 0, 60000, 150000),
    ("fp64", 1, 0.2, 0, 30000, 150000), ("fp64", 2, 0.2, 0, 100000, 320000), ("fp64", 4, 0.2, 0, 200000, 320000),
    ("fp64", 1, 0.3, 0, 0, 320000), ("fp64", 2, 0.3, 0, 200000, 320000), ("fp64", 4, 0.3, 0, 200000, 320000),
    ("fp64", 1, 0.4, 0, 200000, 320000), ("fp64", 2, 0.4, 0, 200000, 320000), ("fp64", 4, 0.4, 0, 260000, 320000),
    ("fp64", 1, 0.5, 0, 200000, 320000), ("fp64", 2, 0.5, 0, 260000, 320000),
    ("fp64 ext", 1, 0.2, 0, 100000, 320000), ("fp64 ext", 2, 0.2, 0, 200000, 320000),
    ("fp64 ext", 4, 0.2, 0, 260000, 320000), ("fp64 ext", 1, 0.3, 0, 260000, 320000),
    ("fp64 ext", 2, 0.3, 0, 260000, 320000), ("fp64 relative", 1, 0.0005, 0, 200000, 320000),
    ("fp64 ext", 1, 0.5, 0, 260000, 320000), ("fp64 relative", 1, 0.0001, 0, 0, 320000),
    ("fp64", 1, 0.2, 300000, 75000, 250000), ("fp64", 1, 0.1, 700000, 60000, 170000),
    ("fp64", 1, 0.2, 700000, 60000, 170000), ("fp64", 1, 0.2, 3000000, 0, 260000),
    ("fp64", 2, 0.2, 3000000, 0, 450000), ("fp64", 4, 0.2, 3000000, 0, 550000),
    ("fp64", 8, 0.2, 3000000, 320000, 640000), ("fp64", 1, 0.3, 3000000, 200000, 550000),
    ("fp64", 2, 0.3, 3000000, 200000, 640000), ("fp64", 1, 0.4, 3000000, 350000, 640000),
    ("fp64 newton", 1, 0.2, 0, 32000, 100000), ("fp64 newton", 4, 0.2, 0, 60000, 150000),
    ("fp64 newton", 1, 0.3, 0, 60000, 100000), ("fp64 newton", 4, 0.3, 0, 60000, 150000),
    ("fp64 newton", 1, 0.5, 0, 60000, 150000), ("fp64 newton ext", 1, 0.2, 0, 60000, 150000),
    ("fp64 newton", 1, 0.2, 1000000, 0, 75000), ("fp64 newton", 8, 0.2, 1000000, 0, 110000),
    ("fp64 newton", 1, 0.3, 1000000, 0, 110000), ("fp64 newton", 8, 0.3, 1000000, 75000, 150000),
    ("fp64 newton", 1, 0.5, 1000000, 110000, 220000), ("fp64 newton", 8, 0.5, 1000000, 110000, 220000),
    ("fp64 newton", 1, 0.8, 1000000, 150000, 250000),
]

SOURCE = """
#include "og_lines.h"
#include <cstdio>
int main() {
  int fp64, newton, ext, relative, leaf;
  double theta, alpha;
  unsigned n;
  while (scanf("%d %d %d %d %d %lf %lf %u", &fp64, &newton, &ext, &relative, &leaf, &theta, &alpha, &n) == 8)
    printf("%u\\n", og::eight_lane_line(og::WalkShape{fp64 != 0, newton != 0, ext != 0, relative != 0, leaf, theta, alpha},
                                       n > 0, n));
}
"""


@pytest.fixture(scope="module")
def line(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("lines")
    (d / "lines.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(d / "lines"), str(d / "lines.cpp")], check=True)

    def ask(rows):
        out = subprocess.run([str(d / "lines")], input="\n".join(rows), capture_output=True, text=True, check=True)
        return [int(v) for v in out.stdout.split()]
    return ask


def _row(kind, leaf, opening, n):
    rel = "relative" in kind
    return "%d %d %d %d %d %g %g %d" % ("fp64" in kind, "newton" in kind, rel or "ext" in kind, rel, leaf,
                                        0.5 if rel else opening, opening if rel else 0.0, n)


def test_line_lies_between_the_measured_times(line):
    lines = line([_row(*m[:4]) for m in MEASURED])
    assert len(lines) == len(MEASURED)
    wrong = [(m, v) for m, v in zip(MEASURED, lines) if not m[4] <= v < m[5]]
    assert not wrong, wrong


def test_line_over_the_whole_range(line):
    """Never above twice the whole-box line, at least that of small theta and
    leaves, and monotone in theta and leaf size."""
    for kind, most in (("mixed", 160000), ("fp64", 320000), ("mixed newton", 70000), ("fp64 newton", 150000)):
        for n in (0, 100, 10 ** 6, 10 ** 8):
            rows = [(leaf, t) for leaf in (1, 2, 3, 8, 4096) for t in (0.0, 0.15, 0.2, 0.4, 0.45, 0.5, 1.0, 5.0)]
            got = dict(zip(rows, line([_row(kind, leaf, t, n) for leaf, t in rows])))
            for (leaf, t), v in got.items():
                assert 0 <= v <= (2 * most if n else most)
                assert v <= got[4096, t] and v <= got[leaf, 5.0]
            assert got[8, 0.5] >= most
