"""Registers of the built kernels, from the notes of the library's code objects: none keeps more than two of them in memory.
Needs no GPU."""
import os
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 images of a library's offload bundles."""
    data = open(path, "rb").read()
    for at in (m.start() for m in re.finditer(MAGIC, data)):
        count, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in name:
                yield data[at + offset:at + offset + size]


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_spilled_registers(tmp_path):
    from paper_2506_02024_amd import build

    if build.is_stale():
        build.build_library()
    spills = {}
    for i, image in enumerate(code_objects(build.lib_path())):
        path = tmp_path / ("image%d.o" % i)
        path.write_bytes(image)
        notes = subprocess.run([READELF, "--notes", str(path)], stdout=subprocess.PIPE, text=True, check=True).stdout
        for kernel in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
            spills[name] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
    assert sum("nested_rows_kernel" in name for name in spills) >= 11
    # 256 x 256 tiles of the register path have 256 accumulators and fragments in 256 registers: two of their addresses lie in memory.  The store to
    # rows that start anywhere, beside a second way to store rows, once made it six in the kernel of most FP16 prefills.
    worst = {name: n for name, n in spills.items() if n > 2}
    assert not worst, worst
