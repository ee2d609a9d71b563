"""How the tiled GEMMs store Y (csrc/gemm_plan.h: store_kind): the rule, asked on the CPU, and each kind on the GPU inside and at the
edges of tiles, with and without a bias, at an address that is not a line's.  The bytes around Y stay as they were."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from gpu_util import CSRC, codes4_to_dev, codes8_to_dev

KINDS = ("cached", "through", "past")


def store_kinds(questions, tmp_path):
    """(bits, M, N, K, address of Y) -> kind"""
    src, exe = tmp_path / "kind.cpp", str(tmp_path / "kind")
    src.write_text('#include "gemm_plan.h"\n#include <cstdio>\nusing namespace convrot::gemm;\nint main() {\n  long b, M, N, K, y;\n'
                   '  while (std::scanf("%ld %ld %ld %ld %ld", &b, &M, &N, &K, &y) == 5)\n'
                   '    std::printf("%d\\n", (int)(b == 4 ? store_kind<4>(choose<4>(M, N, K), M, N, K, y) : store_kind<8>(choose<8>(M, N, K), M, N, K, y)));\n}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(src)], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, input="\n".join(" ".join(map(str, q)) for q in questions)).stdout.split()
    return [KINDS[int(o)] for o in out]


# (M, N, K), bytes from a line's start to Y, kinds at 4 and 8 bits
CASES = [((300, 320, 96), 0, "through", "through"), ((4609, 1280, 1056), 0, "through", "through"), ((515, 3080, 1056), 0, "through", "through"),
         ((1030, 1088, 544), 16, "through", "through"), ((4100, 4360, 192), 0, "cached", "cached"), ((2300, 7744, 160), 112, "cached", "cached"),
         ((5082, 6320, 768), 0, "cached", "through"), ((3001, 3070, 160), 0, "cached", "cached"), ((4000, 2136, 7200), 0, "cached", "cached"), ((4000, 2136, 3200), 0, "through", "through"), ((3100, 2304, 2048), 0, "through", "past"),
         ((7700, 6272, 160), 0, "cached", "cached"), ((7600, 6272, 160), 0, "through", "through"), ((4100, 4096, 4096), 0, "past", "past"), ((5001, 12224, 1056), 0, "past", "past")]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_rule(tmp_path):
    questions = [(bits, *s, 4096 + off) for s, off, _, _ in CASES for bits in (4, 8)]
    assert store_kinds(questions, tmp_path) == [k for c in CASES for k in c[2:]]
    # no half line and no short product goes past the caches, whatever its size; the benchmark's long layers do
    q = [(bits, M, N, K, y) for bits in (4, 8) for M in (1, 77, 512, 4608, 16896, 2 ** 31 - 1) for N in (64, 1000, 3072, 12264, 12288, 2 ** 31 - 64)
         for K in (32, 64, 512, 3072, 15360, 65536) for y in (0, 16, 64, 128)]
    for (bits, M, N, K, y), kind in zip(q, store_kinds(q, tmp_path)):
        if kind == "past":
            assert N % 64 == 0 and y % 128 == 0 and M * N * K >= (1.5e10 if bits == 4 else 7.5e9) and K >= 512, (bits, M, N, K, y)
    long = [(4, 4608, 3072, 3072, 0), (4, 4608, 12288, 3072, 0), (4, 4608, 3072, 12288, 0), (4, 16896, 3072, 12288, 0), (8, 4608, 12288, 3072, 0)]
    assert store_kinds(long, tmp_path) == ["past"] * 5


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}+{c[1]}")
def test_stored_rows(case, bits):
    from paper_2512_03673_amd import binding as cr
    (M, N, K), off, _, _ = case
    print(f"bits={bits} M={M} N={N} K={K} offset {off}", flush=True)
    rng = np.random.default_rng(M + N + K + off)
    top = 7 if bits == 4 else 127
    qx, qw = (rng.integers(-top, top + 1, (r, K), dtype=np.int8) for r in (M, N))
    to_dev, gemm = (codes4_to_dev, cr.convrot_w4a4_gemm_dequant) if bits == 4 else (codes8_to_dev, cr.convrot_w8a8_gemm_dequant)
    Xq, Wq = to_dev(qx), to_dev(qw)
    sx, sw = (torch.from_numpy(rng.uniform(0.5, 2.0, r).astype(np.float32)).cuda() for r in (M, N))
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32) * 50).cuda().to(torch.bfloat16)
    # whole numbers below 2^53: the product in doubles is exact
    t = (torch.from_numpy(qx).cuda().double() @ torch.from_numpy(qw).cuda().double().T) * sx.double()[:, None] * sw.double()
    buf = torch.empty(M * N + 256, dtype=torch.bfloat16, device="cuda")
    assert buf.data_ptr() % 128 == 0
    y = buf[64 + off // 2:64 + off // 2 + M * N].view(M, N)
    for b in (None, bias):
        buf.fill_(3.0)
        gemm(Xq, sx, Wq, sw, K, Y=y, bias=b)
        torch.cuda.synchronize()
        ref = t if b is None else t + b.double()
        # one rounding to bf16 (2^-8 of the value at most) of a value that took three fp32 roundings of t and t + b
        bound = ref.abs() * (2.0 ** -8 * (1 + 2.0 ** -20)) + (t.abs() + ref.abs()) * 2.0 ** -22
        assert ((y.double() - ref).abs() <= bound).all()
        assert (buf[:64 + off // 2] == 3.0).all() and (buf[64 + off // 2 + M * N:] == 3.0).all()
