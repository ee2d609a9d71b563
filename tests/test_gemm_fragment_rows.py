"""Which rows the 16-row fragments of the tiled GEMM take (csrc/fragment_rows.h): a pair covers its 32 rows once, a lane of the result has two neighbouring
columns, and reads meet on no LDS bank; then products of few stages, whose first and last ones take other ways through the loop: of every tile with each number of
stages up to two more than its ring holds, as far as the plan gives it such (not 256 x 256 and 128 x 192 at 4 bits, which it takes from eight and seven stages on)."""
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


# bits, tile: stages of its ring; shapes of 1, 2, ... stages up to two more than that.  (128 x 128 at 4 bits: up to 256 tiles, and more.)
FEW = {
    (4, "192x192"): (2, [(657, 10988, 128), (641, 10961, 160), (646, 10916, 384), (641, 11226, 480)]),
    (4, "256x128"): (2, [None, (1163, 9806, 192), (1281, 8837, 384), (1285, 8900, 480)]),
    (4, "256x128w8"): (3, [None, (386, 11809, 192), (390, 9423, 288), (327, 11077, 416), (323, 11281, 544)]),
    (4, "128x128"): (4, [(261, 9854, 96), (262, 9958, 224), (131, 11004, 352), (129, 11043, 448), (132, 10907, 544), (132, 11051, 736)]),
    (4, "128x128", "many"): (3, [(397, 11657, 64), (515, 9336, 192), (515, 11055, 320), (518, 10945, 416), (524, 10906, 544)]),
    (4, "64x64"): (3, [(33, 4147, 32), (300, 2050, 160), (300, 2050, 320), (4110, 66, 448), (300, 2050, 576)]),
    (8, "64x64"): (4, [(33, 4147, 32), (300, 2050, 96), (300, 2050, 160), (4305, 65, 224), (300, 2050, 288), (300, 2050, 384)]),
    (8, "128x128"): (4, [(131, 11054, 32), (129, 10890, 96), (134, 10883, 160), (131, 10934, 256), (129, 11630, 320), (131, 11004, 352)]),
    (8, "192x192"): (3, [None, (643, 12028, 96), (653, 11932, 192), (641, 11013, 224), (641, 11163, 288)]),
    (8, "256x128"): (3, [None, None, (1163, 9806, 192), (1025, 11309, 224), (1167, 9796, 288)]),
    (8, "128x192"): (3, [(397, 11657, 64), (398, 11652, 128), (331, 10953, 160), (325, 11271, 256), (390, 9423, 288)]),
}


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
@pytest.mark.parametrize("tile", FEW)
def test_tiles_of_few_stages(tile):
    ring, shapes = FEW[tile]
    assert len(shapes) == ring + 2
    for stages, s in enumerate(shapes, 1):
        if s is None:
            continue
        M, N, K = s
        assert -(-K // (128 if tile[0] == 4 else 64)) == stages and gemm_plans([s])[s][tile[0] == 8] == tile[1], s
        if tile[:2] == (4, "128x128"):
            assert (-(-M // 128) * -(-N // 128) > 256) == (len(tile) == 3)


@pytest.mark.gpu
@pytest.mark.parametrize("tile", FEW)
def test_first_refills(tile):
    """Less than the ring holds, as much, and the first stages that refill it."""
    for s in FEW[tile][1]:
        if s is not None:
            M, N, K = s
            print(f"{tile} M={M} N={N} K={K}", flush=True)
            check_product(tile[0], M, N, K, np.unique(np.concatenate([np.arange(0, M, 61), np.arange(max(M - 33, 0), M)])))
