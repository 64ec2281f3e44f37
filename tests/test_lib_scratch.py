"""Scratch memory per lane of the kernels in the built library, from the code
objects' own metadata.  The cost and guidance kernels are fast where they keep
their state in registers: with the frames' tables kept in scratch across the
swept samples (336 bytes per lane) a gradient with eight of them took 1.6 times
as long."""
import os
import re
import struct
import subprocess

import pytest

from paper_2410_16727_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
if not (os.path.exists(build.LIB) and os.path.exists(READELF)):
    pytest.skip("needs the built library and llvm-readelf", allow_module_level=True)

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects():
    """The gfx950 code objects of every translation unit."""
    data = open(build.LIB, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, pos - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            if b"gfx950" in data[pos + 24:pos + 24 + n] and size:
                yield data[at + off:at + off + size]
            pos += 24 + n
        at = data.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """Mangled kernel name -> bytes per lane."""
    got = {}
    path = str(tmp_path_factory.mktemp("obj") / "code.o")
    for obj in code_objects():
        with open(path, "wb") as f:
            f.write(obj)
        notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
        names = re.findall(r"^\s*\.name:\s+(_Z\w+)$", notes, re.M)
        sizes = re.findall(r"^\s*\.private_segment_fixed_size:\s+(\d+)$", notes, re.M)
        assert len(names) == len(sizes)
        got.update(zip(names, map(int, sizes)))
    return got


@pytest.mark.parametrize("kernel", ["k_cost", "k_guide"])
@pytest.mark.parametrize("terms,full,most", [(0, 0, 0), (0, 1, 0), (1, 1, 0), (1, 0, 240)])
def test_cost_kernels(scratch, kernel, terms, full, most):
    """(template arguments: optional terms, full team)"""
    found = [v for k, v in scratch.items() if f"{kernel}ILb{terms}ELb{full}E" in k]
    assert len(found) == 1 and found[0] <= most, (kernel, terms, full, found)
