"""Every tile of a GEMM's grid is some block's, and no tile two blocks' (csrc/gemm_plan.h, where a block divides by multiplying with reciprocals)."""
import os
import shutil
import subprocess

import pytest

from gpu_util import CSRC, gemm_plans

SOURCE = r"""
#include "gemm_plan.h"
#include <cstdio>
#include <random>
#include <vector>
using namespace convrot::gemm;

static int grid(int tiles_m, int tiles_n, int rows)
{
    const TileOrder o = tile_order(tiles_m, tiles_n, rows);
    std::vector<int> seen((size_t)tiles_m * tiles_n);
    for (int xcd = 0; xcd < kNumXcd; ++xcd) {
        int last_band = 0;
        for (int turn = 0; turn < o.per_xcd + 9; ++turn) {
            int tm = -1, tn = -1;
            if (!tile_of_block(o, turn * kNumXcd + xcd, tm, tn) || tn >= tiles_n) continue;
            const int id = xcd * o.per_xcd + turn, band = id / (rows * tiles_n), first = band * rows;
            const int high = tiles_m - first < rows ? tiles_m - first : rows, local = id - band * rows * tiles_n;
            if (tm != first + local % high || tn != local / high || band < last_band) return 1;
            last_band = band;
            if (seen[(size_t)tm * tiles_n + tn]++) return 2;
        }
    }
    for (int n : seen) if (n != 1) return 3;
    return 0;
}

int main()
{
    for (int m = 1; m <= 40; ++m)
        for (int n = 1; n <= 40; ++n)
            for (int rows : {4, 6, 8})
                if (const int e = grid(m, n, rows)) { std::printf("%d x %d in bands of %d: %d\n", m, n, rows, e); return 1; }
    for (auto [m, n] : {std::pair{1, 100003}, {100003, 1}, {7, 65537}, {65537, 9}, {1000, 1001}})
        for (int rows : {4, 6, 8})
            if (const int e = grid(m, n, rows)) { std::printf("%d x %d in bands of %d: %d\n", m, n, rows, e); return 1; }
    std::mt19937 gen(1);
    for (int i = 0; i < 3000000; ++i) {
        const int d = 1 + (int)(gen() >> (3 + gen() % 29)), k = (int)(gen() >> (5 + gen() % 27)) / d;
        for (int n : {k * d - 1, k * d, k * d + 1, (int)(gen() >> 5)})
            if (n >= 0 && divide(n, d, reciprocal(d)) != n / d) { std::printf("%d / %d\n", n, d); return 1; }
    }
    std::puts("ok");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_blocks_and_tiles_are_one_to_one(tmp_path):
    (tmp_path / "order.cpp").write_text(SOURCE)
    exe = str(tmp_path / "order")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(tmp_path / "order.cpp")], check=True)
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.stdout.strip() == "ok", run.stdout


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_no_block_takes_a_tile_outside_the_widest_outputs(tmp_path):
    # One row of 192-column tiles (M up to 192) up to the widest output whose tiles are counted in 32 bits: a tile past the last one starts
    # past 2^31 columns there.
    (tmp_path / "wide.cpp").write_text("""
#include "gemm_plan.h"
#include <cstdio>
#include <initializer_list>
using namespace convrot::gemm;
int main()
{
    for (int N : {2147483136, 2147483137, 2147483300, 2147483456, 1073741825, 191, 193}) {
        const int tiles = (N + 191) / 192;
        const TileOrder o = tile_order(1, tiles, 8);
        int inside = 0, outside = 0;
        for (int bid = (o.per_xcd > 9 ? o.per_xcd - 9 : 0) * kNumXcd; bid < (o.per_xcd + 9) * kNumXcd; ++bid) {
            int tm = -1, tn = -1;
            if (!tile_of_block(o, bid, tm, tn)) continue;
            (starts_inside(tn, 192, N) ? inside : outside)++;
            if (tm != 0 || starts_inside(tn, 192, N) != (tn < tiles)) { std::printf("N %d: tile %d\\n", N, tn); return 1; }
        }
        if (outside != o.per_xcd * kNumXcd - tiles || inside < 1) { std::printf("N %d: %d outside\\n", N, outside); return 1; }
    }
    std::puts("ok");
}
""")
    exe = str(tmp_path / "wide")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(tmp_path / "wide.cpp")], check=True)
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.stdout.strip() == "ok", run.stdout
    # ... and such products are 192 columns wide
    widest = [(1, 2147483300, 32), (192, 2147483137, 64), (1, 2147483456, 128)]
    assert {p.split("x")[1] for plans in gemm_plans(widest).values() for p in plans} == {"192"}
