"""The line between the mesh deposit by atomics and by blocks against measured
times of the whole call (host only: the rule is plain C++)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_17658_amd", "csrc")

# (mesh, particles, atomics us, blocks us): particles in grid order, whose atomics
# are cheapest, and clustered ones in random order
MEASURED = [
    (128, 97336, 187, 223), (128, 262144, 213, 237), (128, 1000000, 263, 259), (128, 1331000, 283, 279),
    (128, 700000, 780, 355), (128, 1350000, 1350, 470), (256, 262144, 898, 948), (256, 343000, 912, 966),
    (256, 729000, 988, 1000), (256, 1000000, 1032, 1018), (256, 2097152, 1156, 1103), (256, 100000, 865, 939),
    (256, 700000, 1227, 1072), (256, 2000000, 1953, 1347), (512, 512000, 7961, 8419), (512, 1000000, 8123, 8524),
    (512, 2097152, 8378, 8682), (512, 500000, 8005, 8512), (512, 1000000, 8322, 8642), (512, 1350000, 8539, 8746)]


def test_line(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    (tmp_path / "line.cpp").write_text('#include "og_lines.h"\n#include <cstdio>\nint main() {\n  unsigned n;\n'
                                       '  while (scanf("%u", &n) == 1) printf("%llu\\n", '
                                       '(unsigned long long)og::block_deposit_line(n));\n}\n')
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(tmp_path / "line"), str(tmp_path / "line.cpp")], check=True)
    out = subprocess.run([str(tmp_path / "line")], input=" ".join(str(m[0]) for m in MEASURED), capture_output=True,
                         text=True, check=True).stdout.split()
    for (mesh, n, atomics, blocks), line in zip(MEASURED, out):
        if n >= int(line):  # by blocks: at most 2 % slower
            assert blocks <= 1.02 * atomics, (mesh, n, line)


def test_sort_of_half_a_million_keys_fills_the_chip():
    """Around the line the sort by blocks has at least a workgroup per compute
    unit (256): with 4096 keys each it had 122, and the call was slower than the
    atomics for particles in grid order."""
    def constant(name, source):
        text = open(os.path.join(CSRC, source)).read()
        return int(text.split("constexpr uint32_t %s = " % name)[1].split(";")[0])
    tile, small = constant("kSortTile", "og_kernels.h"), constant("kSmallTiles", "k_pm.hip")
    assert 500000 <= small
    for n in (500000, small, small + 1, 2097152):
        assert -(-n // (tile // 4 if n <= small else tile)) >= 256, n
