"""The one-launch forward at the edges of its block widths (16, 32, 48 and 64 columns): the last output width of each, the
first of the next, ragged last blocks."""
import pytest

import test_forward_small


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("M,N,K", [(1, 4097, 96), (3, 8193, 1024), (1, 8199, 3072), (8, 8192, 160), (2, 12288, 1056), (4, 12289, 64), (2, 12291, 2048), (3, 16383, 544)])
def test_one_launch_equals_two(M, N, K, bits):
    test_forward_small.test_one_launch_equals_two(M, N, K, bits)
