"""The one-launch forward in tiles of rows against the two launches it stands for: same codes, scales and output, bit for bit, at the
edges of its tiles: rows that do not divide among them or among the code layouts' blocks of 16 and 32, one to four stretches of 1024
elements a row, each block width, ragged N and K.  Which shapes those are is a host function, asked on the CPU."""
import shutil
import subprocess

import pytest

import test_forward_small
from gpu_util import CSRC

# (M, N, K): (rows, columns) of a block
SHAPES = {(9, 64, 256): (9, 32), (17, 33, 32): (9, 32), (31, 1000, 96): (16, 32), (33, 500, 1024): (11, 32), (256, 1024, 1024): (16, 64), (250, 512, 320): (16, 32),
          (257, 960, 1024): (16, 64), (100, 1537, 1056): (8, 128), (389, 437, 1056): (8, 128), (40, 6100, 1024): (14, 128), (4096, 77, 1024): (16, 128),
          (25, 513, 2048): (7, 32), (13, 700, 2080): (5, 32), (6, 90, 4096): (3, 32), (3, 5000, 160): (3, 32), (16, 8192, 1280): (8, 64), (11, 8191, 1280): (6, 64)}
SHAPES8 = [s for s, (_, columns) in SHAPES.items() if s[2] * columns * 2 <= 144 * 1024]
OTHERS = [(4097, 64, 64), (256, 2049, 1024), (389, 437, 1312), (257, 1000, 2048), (60, 1024, 3072), (1, 32769, 32), (2, 64, 4128), (2 ** 31 - 1, 2 ** 31 - 1, 65536)]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_which_shapes_take_row_tiles(tmp_path):
    src = tmp_path / "rule.cpp"
    src.write_text('#include "gemm_plan.h"\n#include <cstdio>\n#include <cstdlib>\nusing namespace convrot::gemm;\nint main(int n, char **v) {\n'
                   '  for (int i = 1; i + 2 < n; i += 3) {\n    const long M = atol(v[i]), N = atol(v[i + 1]), K = atol(v[i + 2]);\n'
                   '    const bool four = forward_in_row_tiles(M, N, K, 4);\n    const RowTiles t = four ? forward_row_tiles(M, N, K) : RowTiles{0, 0};\n'
                   '    std::printf("%d %d %d %d\\n", four, forward_in_row_tiles(M, N, K, 8), t.rows, t.columns);\n  }\n}\n')
    exe = str(tmp_path / "rule")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(src)], check=True)
    many = [(M, N, K) for M in (1, 2, 5, 15, 16, 17, 100, 255, 1000, 4096) for N in (1, 31, 32, 33, 64, 1000, 8192, 32768) for K in (32, 1024, 1056, 2048, 2080, 3104, 4096)]
    shapes = list(SHAPES) + OTHERS + many
    out = subprocess.run([exe] + [str(d) for s in shapes for d in s], check=True, capture_output=True, text=True).stdout.split()
    got = {s: tuple(int(o) for o in out[4 * i:4 * i + 4]) for i, s in enumerate(shapes)}
    for s, tile in SHAPES.items():
        assert got[s] == (1, int(s in SHAPES8), *tile), s
    for s in OTHERS:
        assert got[s][:2] == (0, 0), s
    for (M, N, K), (four, eight, rows, columns) in got.items():      # what the kernel is built for
        assert four or not eight
        if four:
            assert 1 <= rows <= 16 and rows * -(-K // 1024) <= 16 and columns in (32, 64, 128) and -(-M // rows) * -(-N // columns) <= 256


@pytest.mark.gpu
@pytest.mark.parametrize("bits,M,N,K", [(4, *s) for s in SHAPES] + [(8, *s) for s in SHAPES8])
def test_one_launch_equals_two(bits, M, N, K):
    test_forward_small.test_one_launch_equals_two(M, N, K, bits)
