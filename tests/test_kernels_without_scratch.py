"""No kernel of the library keeps registers in memory: the built library's own code objects say how much of it a lane has."""
import re
import shutil
import struct
import subprocess

import pytest

from paper_2512_03673_amd import build

READELF = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data: bytes):
    at = data.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, at + len(MAGIC))[0]):
            offset, size, name = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + name]:
                yield data[at + offset:at + offset + size]
            p += 24 + name
        at = data.find(MAGIC, at + 1)


@pytest.mark.skipif(READELF is None, reason="no llvm-readelf")
def test_no_kernel_has_scratch(tmp_path):
    with open(build.LIB, "rb") as f:
        objects = list(code_objects(f.read()))
    found = {}
    for i, o in enumerate(objects):
        (tmp_path / f"{i}.co").write_bytes(o)
        notes = subprocess.run([READELF, "--notes", str(tmp_path / f"{i}.co")], check=True, capture_output=True, text=True).stdout
        for kernel in notes.split(".agpr_count:")[1:]:
            name, bytes_, spills = (re.search(rf"\.{k}:\s+(\S+)", kernel).group(1) for k in ("name", "private_segment_fixed_size", "vgpr_spill_count"))
            found[name] = int(bytes_), int(spills)
    assert len(objects) >= 4 and len(found) > 300 and any("gemm_cut_kernel" in k for k in found)
    assert not {k: v for k, v in found.items() if any(v)}
