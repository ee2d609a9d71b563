"""64 x 64 tiles at 4 bits in a launch of one round, whose ring has four stages from 16 stages of 128 codes on (csrc/gemm_plan.h: deep_ring),
and around that line: ragged edges, a padded last stage, the most tiles of a round and more.  Accumulators bit for bit against the exact
integer product of the same codes, outputs against it dequantised."""
import shutil

import numpy as np
import pytest
import torch

import oracle
from gpu_util import bf16_to_host_bits, bf16_ulp_diff, codes4_to_dev, gemm_plans

SHAPES = [(700, 1000, 2048), (689, 1001, 1952), (255, 3070, 3072), (1024, 1024, 2080), (190, 4090, 2176), (641, 1000, 1920), (1025, 1024, 2080), (512, 3072, 2176)]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_shapes_take_64x64_on_both_sides_of_the_line():
    plans = gemm_plans(SHAPES)
    assert {plans[s][0] for s in SHAPES} == {"64x64"}, plans
    tiles = [-(-M // 64) * -(-N // 64) for M, N, _ in SHAPES]
    deep = [t <= 256 and -(-K // 128) >= 16 for t, (_, _, K) in zip(tiles, SHAPES)]
    assert any(deep) and not all(deep) and 256 in tiles and max(tiles) > 256


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_deep_ring(M, N, K):
    from paper_2512_03673_amd import binding as cr
    print(f"M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(M + N + K)
    qx, qw = (rng.integers(-7, 8, (r, K), dtype=np.int8) for r in (M, N))
    sx, sw = (rng.uniform(0.5, 2.0, r).astype(np.float32) for r in (M, N))
    Xq, Wq = codes4_to_dev(qx), codes4_to_dev(qw)
    acc = cr.convrot_w4a4_gemm_i32(Xq, Wq, M, N, K)
    y = cr.convrot_w4a4_gemm_dequant(Xq, torch.from_numpy(sx).cuda(), Wq, torch.from_numpy(sw).cuda(), K)
    torch.cuda.synchronize()
    ref = (torch.from_numpy(qx).cuda().double() @ torch.from_numpy(qw).cuda().double().T).round().int()      # exact: whole numbers below 2^53
    assert torch.equal(acc, ref)
    assert bf16_ulp_diff(bf16_to_host_bits(y), oracle.dequant(ref.cpu().numpy(), sx, sw)).max() <= 1
