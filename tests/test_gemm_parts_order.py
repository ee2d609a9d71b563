"""The last tiles of some products are cut into parts, which every other XCD begins with (csrc/gemm_plan.h: parts_first, cut_turn): every tile is a block's
once, or each of its parts, in either order; and products on both sides of the line against the exact product."""
import shutil
import subprocess

import numpy as np
import pytest

from gpu_util import CSRC, check_product, gemm_plans

SOURCE = r"""
#include "gemm_plan.h"
#include <cstdio>
#include <vector>
using namespace convrot::gemm;
int main()
{
    constexpr Store past = Store::kPast;
    static_assert(parts_first(past, 1793, 26) && !parts_first(past, 12288, 27) && parts_first(past, 1792, 17) && !parts_first(past, 1792, 18), "lines");
    static_assert(!parts_first(Store::kCached, 12288, 8) && !parts_first(Store::kThrough, 12288, 8), "stores");
    for (int per = 32; per < 5 * 32; ++per) {
        const int parts = parts_of_last_tiles(per);
        if (parts == 1) continue;
        const int whole = per - per % 32, grid = whole + per % 32 * parts;
        if (whole >= kPartsFirst) return 1;
        for (int how : {whole, whole | kPartsFirst})
            for (int xcd = 0; xcd < kNumXcd; ++xcd) {
                std::vector<int> seen(per * parts);
                for (int turn = 0; turn < grid; ++turn) {
                    const CutTurn t = cut_turn(turn, xcd, per, how, parts);
                    if ((int)t.tile >= per || (int)t.part >= parts || t.whole != ((int)t.tile < whole) || (t.whole && t.part)) return 2;
                    const bool begins = how != whole && xcd % 2;
                    if (t.whole != (begins ? turn >= grid - whole : turn < whole)) return 3;
                    seen[t.tile * parts + t.part]++;
                }
                for (int i = 0; i < per * parts; ++i)
                    if (seen[i] != (i / parts >= whole || i % parts == 0)) return 4;
            }
    }
    std::puts("ok");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_every_tile_or_each_of_its_parts_once(tmp_path):
    (tmp_path / "parts.cpp").write_text(SOURCE)
    exe = str(tmp_path / "parts")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(tmp_path / "parts.cpp")], check=True)
    assert subprocess.run([exe], capture_output=True, text=True).stdout == "ok\n"


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(4100, 4608, 3328), (4100, 4608, 3360), (4360, 4864, 3328), (4360, 4864, 3360),      # quarters, halves; 26 and 27 stages
                                   (15888, 1216, 2176), (15888, 1216, 2208),                                            # narrow: 17 and 18
                                   (4100, 4600, 3328), (4100, 4600, 3360), (4360, 4870, 3328), (4360, 4870, 3360)])     # rows that are not whole lines
def test_both_orders(M, N, K):
    assert gemm_plans([(M, N, K)])[(M, N, K)][0] == "256x256" and 32 < (-(-M // 256) * -(-N // 256) + 7) // 8 <= 48
    print(f"M={M} N={N} K={K}", flush=True)
    check_product(4, M, N, K, np.unique(np.concatenate([np.arange(0, M, 61), [M - 1]])))
