"""The tiles that take a ring of four stages in a launch of one round: both sides of the number of stages from which they do (16 of
128 codes, 16 of 64), one tile more than a round, whole and ragged edges, the last stage padded.  Accumulators bit for bit
against the exact integer product of the same codes, outputs against it dequantised."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import bf16_to_host_bits, bf16_ulp_diff, codes4_to_dev, codes8_to_dev, gemm_plans

SHAPES = [(4, 3000, 2900, 2048), (4, 2881, 3072, 1952), (4, 3070, 2876, 2080), (4, 2944, 3001, 3072), (8, 511, 12280, 1024), (8, 511, 12285, 960),
          (8, 509, 12285, 1120), (8, 512, 12281, 3040)]


@pytest.mark.gpu
@pytest.mark.parametrize("bits,M,N,K", SHAPES)
def test_deep_ring(bits, M, N, K):
    from paper_2512_03673_amd import binding as cr
    tile = gemm_plans([(M, N, K)])[(M, N, K)][bits == 8]
    assert tile == ("192x192" if bits == 4 else "128x192")
    print(f"bits={bits} M={M} N={N} K={K} tile {tile}", flush=True)
    rng = np.random.default_rng(M + N + K)
    top = 7 if bits == 4 else 127
    qx, qw = (rng.integers(-top, top + 1, (r, K), dtype=np.int8) for r in (M, N))
    sx, sw = (rng.uniform(0.5, 2.0, r).astype(np.float32) for r in (M, N))
    dev = codes4_to_dev if bits == 4 else codes8_to_dev
    Xq, Wq = dev(qx), dev(qw)
    acc = (cr.convrot_w4a4_gemm_i32 if bits == 4 else cr.convrot_w8a8_gemm_i32)(Xq, Wq, M, N, K)
    y = (cr.convrot_w4a4_gemm_dequant if bits == 4 else cr.convrot_w8a8_gemm_dequant)(Xq, torch.from_numpy(sx).cuda(), Wq, torch.from_numpy(sw).cuda(), K)
    torch.cuda.synchronize()
    # whole numbers below 2^53: the product in doubles is exact
    ref = (torch.from_numpy(qx).cuda().double() @ torch.from_numpy(qw).cuda().double().T).round().int()
    assert torch.equal(acc, ref)
    rows = np.unique(np.concatenate([np.arange(0, M, 97), [M - 1]]))
    d = bf16_ulp_diff(bf16_to_host_bits(y[torch.from_numpy(rows).cuda()]), oracle.dequant(ref.cpu().numpy()[rows], sx[rows], sw))
    assert d.max() <= 1
