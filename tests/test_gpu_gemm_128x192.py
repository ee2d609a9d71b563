"""128 x 192 tiles of 4-bit codes on six wavefronts: as few stages as the plan gives them (seven, a ring of four) and many, ragged and whole edges, one row of
tiles and many, full and not."""
import numpy as np
import pytest

from gpu_util import check_product, gemm_plans

SHAPES = [(600, 9272, 832), (598, 9223, 832), (1080, 5161, 928), (2096, 2717, 928), (873, 6886, 1056), (1575, 3185, 1056), (512, 12288, 2048), (13324, 307, 2528),
          (4731, 965, 2112), (897, 5953, 2016), (2637, 1728, 4320)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_128x192(M, N, K):
    assert gemm_plans([(M, N, K)])[(M, N, K)][0] == "128x192"
    print(f"M={M} N={N} K={K}", flush=True)
    check_product(4, M, N, K, np.unique(np.concatenate([np.arange(0, M, 53), [M - 1]])), bias=True)
