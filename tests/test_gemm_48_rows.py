"""Small products in tiles of 48 x 32 (csrc/gemm_plan.h: rows_of_48): which take them, on the CPU, and on both sides of the lines against the exact product."""
import shutil
import subprocess

import pytest

from gpu_util import CSRC, check_product, gemm_plans

# bits, M, N, K, in tiles of 48 x 32: where these are at most 256 (M 77: N 4096, M 97: N 2720) and tiles of 32 x 32 more (M 48: from N 4097 on); instead of 16 x 32 from 34 stages
# on (one row of tiles 40; at 8 bits 18), with less of them they were slower.
SHAPES = [(8, 77, 3072, 3072, True), (8, 77, 4096, 1056, True), (8, 77, 4097, 1056, False), (8, 96, 2723, 1280, True), (8, 97, 2723, 1280, False), (8, 40, 5056, 2336, True),
          (8, 48, 4129, 15360, True), (8, 32, 4096, 1024, False), (4, 77, 3072, 4096, False), (4, 123, 2240, 3488, True), (4, 48, 4736, 448, True), (4, 49, 4095, 2080, False), (4, 48, 4097, 2080, True),
          (4, 809, 340, 4704, True), (4, 143, 1599, 4512, False), (4, 35, 7104, 768, True), (4, 35, 8200, 768, False),
          (4, 100, 2246, 4224, False), (4, 100, 2246, 4256, True), (4, 33, 5178, 4992, False), (4, 33, 5178, 5024, True), (8, 77, 3200, 1088, False), (8, 77, 3200, 1120, True)]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_rule(tmp_path):
    src, exe = tmp_path / "rule.cpp", str(tmp_path / "rule")
    src.write_text('#include "gemm_plan.h"\n#include <cstdio>\nusing namespace convrot::gemm;\nint main() {\n  long b, M, N, K;\n'
                   '  while (std::scanf("%ld %ld %ld %ld", &b, &M, &N, &K) == 4) std::printf("%d ", (int)(b == 4 ? rows_of_48<4>(choose<4>(M, N, K), M, N, (K + 127) / 128) : rows_of_48<8>(choose<8>(M, N, K), M, N, (K + 63) / 64)));\n}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(src)], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, input="\n".join(" ".join(map(str, s[:4])) for s in SHAPES)).stdout.split()
    assert [bool(int(v)) for v in out] == [s[4] for s in SHAPES]


@pytest.mark.gpu
@pytest.mark.parametrize("bits,M,N,K", [s[:4] for s in SHAPES])
def test_products(bits, M, N, K):
    print(f"bits={bits} M={M} N={N} K={K} plan {gemm_plans([(M, N, K)])[(M, N, K)][bits == 8]}", flush=True)
    check_product(bits, M, N, K, bias=True)
