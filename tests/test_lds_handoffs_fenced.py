"""What a wavefront stores to LDS by plain stores and others read behind a meeting has a fence on either side of the meeting: a bare one orders nothing for the
compiler.  Seen in the compiler's own intermediate form of the 8-bit GEMM, whose tiled and K-splitting kernels are the 4-bit ones' templates."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_03673_amd import build

FENCE = re.compile(r'fence syncscope\("workgroup"\) (release|acquire|acq_rel|seq_cst)')
BARRIER = "@llvm.amdgcn.s.barrier()"
STORE = re.compile(r"\bstore .*ptr addrspace\(3\)")
LOAD = re.compile(r"= load .*ptr addrspace\(3\)")


def unfenced(body: str):
    """Meetings behind plain stores to LDS, without a release between, and the first loads from LDS behind such meetings without an acquire."""
    stored = handed = False
    for line in body.splitlines():
        if FENCE.search(line):
            kind = FENCE.search(line).group(1)
            stored = stored and kind == "acquire"
            handed = handed and kind == "release"
        elif STORE.search(line):
            stored = True
        elif BARRIER in line:
            if stored:
                yield line
            handed, stored = handed or stored, False
        elif LOAD.search(line) and handed:
            yield line


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_plain_stores_are_fenced(tmp_path):
    out = str(tmp_path / "gemm.ll")
    subprocess.run(["hipcc", *build.FLAGS, "--offload-device-only", "-S", "-emit-llvm", "-o", out, os.path.join(build.CSRC, "gemm_w8a8.hip")], check=True,
                   capture_output=True)
    with open(out) as f:
        kernels = re.findall(r"^define [^@]*amdgpu_kernel [^@]*@(\S+?)\(.*?\{\n(.*?)^\}", f.read(), re.S | re.M)
    assert len(kernels) >= 20 and any("gemm_tiled" in name for name, _ in kernels)
    assert any(STORE.search(body) and FENCE.search(body) and BARRIER in body for _, body in kernels)
    assert not [name for name, body in kernels if any(unfenced(body))]
