"""Registers of the built walk kernels, read from the library's own code objects:
how many waves share a SIMD follows from them (512 vector registers a SIMD, in
blocks of 8), and a register held through a walk's loop for the sake of the
group queue costs some kernels a wave or spills (host only)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2609_17658_amd import og

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled kernel: (vector registers, spilled vector registers)}"""
    if not os.path.exists(READELF) or not shutil.which("c++filt"):
        pytest.skip("no llvm-readelf or c++filt")
    data = open(og.LIB_PATH, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    out, at = {}, data.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        entry = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, entry)
            name = data[entry + 24:entry + 24 + length]
            entry += 24 + length
            if b"gfx950" not in name:
                continue
            elf = tmp_path_factory.mktemp("code") / "code.elf"
            elf.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(elf)], capture_output=True, text=True, check=True).stdout
            for k in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
                def field(f):
                    return re.search(r"\.%s:\s+(\S+)" % f, k).group(1)
                out[field("name")] = (int(field("vgpr_count")), int(field("vgpr_spill_count")))
        at = data.find(magic, at + 24)
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True, check=True).stdout
    return {re.sub(r"^void |\(og::WalkArgs\)$|og::|\(anonymous namespace\)::", "", d): v
            for d, v in zip(names.split("\n"), out.values())}


# waves per SIMD and spilled registers that each kernel is built for
@pytest.mark.parametrize("name,waves,spills", [
    ("k_walkg32<0, true, false>", 6, 0), ("k_walkg32<0, true, true>", 6, 0),
    ("k_walkg32<2, false, false>", 8, 0), ("k_walk64s<2, false, 4, false>", 7, 1),
    ("k_walk64s<0, false, 4, false>", 7, 2), ("k_walk64s<0, false, 4, true>", 6, 22), ("k_walk64<false, true>", 4, 13),
    ("k_walk8<true, false, false>", 5, 0),
    ("k_walk8<false, false, false>", 5, 0), ("k_walk32<5, 2, false, false, false>", 8, 0),
    ("k_walk32<4, 0, true, true, false>", 8, 0), ("k_walk32<4, 2, false, false, false>", 8, 0)])
def test_waves_and_spills(kernels, name, waves, spills):
    vgprs, spilled = kernels[name]
    assert 512 // (-(-vgprs // 8) * 8) >= waves, (vgprs, spilled)
    assert spilled <= spills


def test_list_depths_are_built(kernels):
    """Every depth that walk_list_cap names has its own walk of each kind of box
    (a depth of 4 is not another one's)."""
    for cap in (4, 5, 8, 16, 32):
        for mode in range(4):
            assert "k_walk32<%d, %d, false, false, false>" % (cap, mode) in kernels
