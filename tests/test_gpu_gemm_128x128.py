"""128 x 128 tiles on eight wavefronts and on four (csrc/gemm_plan.h: four_wavefronts_8), alone on their compute unit and two by two: ragged and whole
edges, a few stages and many.  Accumulators bit for bit against the exact integer product of the same codes, outputs against it dequantised."""
import shutil

import numpy as np
import pytest

from gpu_util import check_product, gemm_plans

# up to 256 tiles / more; one stage, as many as the ring, one more, many; at 8 bits 19 and 20 stages are the two sides of a line
SHAPES = [(4, 341, 9152, 64), (4, 424, 6104, 384), (4, 3428, 1052, 160), (4, 336, 5444, 704), (4, 6370, 448, 2496), (4, 7475, 1307, 96), (4, 4854, 2304, 224),
          (4, 3194, 2424, 96), (4, 11400, 960, 480), (8, 139, 12119, 160), (8, 702, 4580, 384), (8, 285, 8951, 1184), (8, 285, 8951, 1216),
          (8, 285, 8951, 1248), (8, 575, 6336, 1600), (8, 4201, 1536, 192), (8, 4990, 1370, 288), (8, 1615, 5632, 64)]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_no_shape_takes_more_of_them_than_a_launch_has():
    # eight wavefronts a tile, and a HIP launch has fewer than 2^32 threads: what such tiles would not fit takes others (192 x 192 tiles of 256 threads fit here)
    shapes = [(M, N, K) for e in (22, 23, 24) for M, N in ((128, (2 ** e + 5) * 128 - 1), ((2 ** e + 5) * 128 - 1, 128), (2 ** (e - 11) * 128 + 1, 2 ** 18)) for K in (32, 64, 128, 1056)
              if max(M, N) < 2 ** 31 - 255 and -(-M // 192) * -(-N // 192) * 256 < 2 ** 32 - 2048]
    took = gemm_plans(shapes)
    assert len(shapes) > 20
    for (M, N, K), plans in took.items():
        assert "128x128" not in plans or (-(-M // 128) * -(-N // 128) + 7) * 512 < 2 ** 32, (M, N, K, plans)


@pytest.mark.gpu
@pytest.mark.parametrize("bits,M,N,K", SHAPES)
def test_128x128(bits, M, N, K):
    assert gemm_plans([(M, N, K)])[(M, N, K)][bits == 8] == "128x128"
    print(f"bits={bits} M={M} N={N} K={K} tiles {-(-M // 128) * -(-N // 128)}", flush=True)
    check_product(bits, M, N, K, np.unique(np.concatenate([np.arange(0, M, 53), [M - 1]])), bias=True)
