"""No kernel of the built library keeps registers in scratch memory: a spilled vector register is a memory
access in the particle loop, in line with the particles' own."""
import re
import struct
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
LIB = ROOT / "paper_2010_11540_amd" / "libscpic.so"
READELF = Path("/opt/rocm/llvm/bin/llvm-readelf")


def _code_objects(data: bytes):
    """The gfx950 code objects of a host library's offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = data.find(magic)
    while at >= 0:
        pos = at + len(magic)
        (count,) = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in name:
                yield data[at + offset:at + offset + size]
        at = data.find(magic, at + 1)


def test_no_kernel_spills_to_scratch(tmp_path):
    if not READELF.exists():
        pytest.skip("no llvm-readelf")
    if not LIB.exists():
        from paper_2010_11540_amd import build
        build.build()
    kernels = {}
    for k, obj in enumerate(_code_objects(LIB.read_bytes())):
        f = tmp_path / f"{k}.co"
        f.write_bytes(obj)
        notes = subprocess.run([str(READELF), "--notes", str(f)], capture_output=True, text=True,
                               check=True).stdout
        for block in notes.split("- .agpr_count:")[1:]:
            field = lambda key: re.search(rf"\.{key}:\s+(\S+)", block).group(1)
            kernels[field("name")] = (int(field("private_segment_fixed_size")),
                                      int(field("vgpr_spill_count")))
    assert len(kernels) > 50
    spilled = {k: v for k, v in kernels.items() if v != (0, 0)}
    assert not spilled
