"""Which rows the 16-row fragments of the tiled GEMM take (csrc/fragment_rows.h): a pair covers its 32 rows once, a lane of the result has two neighbouring
columns, and reads meet on no LDS bank; then the few-stage products of every tiled kernel, whose first and last stages take other ways through the loop."""
import shutil
import subprocess

import numpy as np
import pytest

from gpu_util import CSRC, _swz_a, _swz_b, check_product, gemm_plans


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_rows_and_banks(tmp_path):
    src, exe = tmp_path / "rows.cpp", str(tmp_path / "rows")
    src.write_text('#include "fragment_rows.h"\n#include <cstdio>\nusing namespace convrot::gemm;\nint main() {\n'
                   '  for (int odd = 0; odd < 2; ++odd) for (int c = 0; c < 16; ++c) std::printf("%d ", row_of(c, odd));\n'
                   '  for (int q = 0; q < 4; ++q) std::printf("%d ", piece_of(q));\n}\n')
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", exe, str(src)], check=True)
    v = [int(x) for x in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()]
    rows, piece = np.array(v[:32]).reshape(2, 16), v[32:]
    assert sorted(rows.ravel()) == list(range(32)) and sorted(piece) == [0, 1, 2, 3]
    assert (rows // 2 == np.arange(16)).all()                # columns 2 c and 2 c + 1 of Y lie in lane c
    lanes = np.arange(64)
    turns128 = [np.r_[0:4, 12:16, 20:28], np.r_[4:12, 16:20, 28:32]]
    turns128 += [t + 32 for t in turns128]
    for odd in (0, 1):
        r, c = rows[odd][lanes % 16], np.array(piece)[lanes // 16]
        s16 = ((r % 16 >> 1) ^ (r % 16 >> 3)) & 3            # 8-bit panels, which are swizzled as they are copied to LDS
        reads = [(16, r * 64 + (c ^ _swz_a(r)) * 16, turns128), (16, r * 64 + (c ^ s16) * 16, turns128),
                 (8, r * 32 + (c ^ _swz_b(r)) * 8, [lanes[:32], lanes[32:]])]
        for width, at, turns in reads:
            for t in turns:
                assert len(set(at[t] // width % (256 // width))) == len(t)       # 64 banks of 4 bytes


SIZES = [(129, 65), (1023, 3070), (2300, 2300), (4601, 3068), (3001, 3070), (4351, 4601)]


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("K", [32, 96, 128, 224, 320, 480, 544, 1056])
def test_few_stages(K, bits):
    """One to nine stages at 4 bits, one to seventeen at 8."""
    plans = gemm_plans([(M, N, K) for M, N in SIZES])
    for M, N in SIZES:
        print(f"bits={bits} M={M} N={N} K={K} tile {plans[(M, N, K)][bits == 8]}", flush=True)
        check_product(bits, M, N, K, np.unique(np.concatenate([np.arange(0, M, 61), np.arange(max(M - 33, 0), M)])))
