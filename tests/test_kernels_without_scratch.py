"""What the built library's own code objects say of its kernels: none keeps registers in memory, and those of rotate+quantise that run fastest with six wavefronts on a SIMD
have more registers than eight would leave them."""
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


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name: (bytes of scratch, registers spilled, registers set aside)}"""
    if READELF is None:
        pytest.skip("no llvm-readelf")
    with open(build.LIB, "rb") as f:
        objects = list(code_objects(f.read()))
    found, at = {}, tmp_path_factory.mktemp("objects")
    for i, o in enumerate(objects):
        (at / f"{i}.co").write_bytes(o)
        text = subprocess.run([READELF, "-W", "--notes", "--sections", "--syms", str(at / f"{i}.co")], check=True, capture_output=True, text=True).stdout
        sections = {n: int(offset, 16) - int(address, 16) for n, address, offset in re.findall(r"^ +\[ *(\d+)\] \S+ +\S+ +([0-9a-f]{16}) ([0-9a-f]{6}) ", text, re.M)}
        # the first six bits of the word at 48 of a kernel's descriptor: registers of a lane in eights, less one
        descriptors = {name: struct.unpack_from("<I", o, sections[n] + int(address, 16) + 48)[0] & 63
                       for address, n, name in re.findall(r": ([0-9a-f]{16}) +64 OBJECT .* (\d+) (\S+)\.kd$", text, re.M)}
        for kernel in text.split(".agpr_count:")[1:]:
            name, *numbers = (re.search(rf"\.{k}:\s+(\S+)", kernel).group(1) for k in ("name", "private_segment_fixed_size", "vgpr_spill_count"))
            found[name] = (*map(int, numbers), 8 * descriptors[name] + 8)
    assert len(objects) >= 4 and len(found) > 300 and any("gemm_cut_kernel" in k for k in found)
    return found


def test_no_kernel_has_scratch(kernels):
    assert not {k: v for k, v in kernels.items() if v[0] or v[1]}


def test_rotate_quantise_leaves_room_for_six_wavefronts(kernels):
    """8-bit codes in rows of 4097 to 8192 elements (U = 2, a row a block), and at g <= 64 of 1025 to 4096 (U = 1, two rows a block): 512 registers of a lane hold seven times 72."""
    rows = {k: v[2] for k, v in kernels.items() if re.search(r"rotquant_kernelILi\d+ELi8ELi2ELi1ELi[34]ELi1EE|rotquant_kernelILi(4|16|64)ELi8ELi1ELi2ELi[234]ELi2EE", k)}
    assert len(rows) == 19 and min(rows.values()) > 72, rows
