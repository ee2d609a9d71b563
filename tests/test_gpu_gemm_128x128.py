"""128 x 128 tiles on eight wavefronts and on four (csrc/gemm_plan.h: four_wavefronts_8), alone on their compute unit and two by two: ragged and whole
edges, a few stages and many.  Accumulators bit for bit against the exact integer product of the same codes, outputs against it dequantised."""
import shutil

import numpy as np
import pytest
import torch

import oracle
from gpu_util import bf16_to_host_bits, bf16_ulp_diff, codes4_to_dev, codes8_to_dev, gemm_plans

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
    from paper_2512_03673_amd import binding as cr
    assert gemm_plans([(M, N, K)])[(M, N, K)][bits == 8] == "128x128"
    print(f"bits={bits} M={M} N={N} K={K} tiles {-(-M // 128) * -(-N // 128)}", flush=True)
    rng = np.random.default_rng(M + N + K)
    top = 7 if bits == 4 else 127
    qx, qw = (rng.integers(-top, top + 1, (r, K), dtype=np.int8) for r in (M, N))
    sx, sw = (rng.uniform(0.5, 2.0, r).astype(np.float32) for r in (M, N))
    dev = codes4_to_dev if bits == 4 else codes8_to_dev
    Xq, Wq = dev(qx), dev(qw)
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32) * 50).cuda().to(torch.bfloat16)
    gemm = cr.convrot_w4a4_gemm_dequant if bits == 4 else cr.convrot_w8a8_gemm_dequant
    scales = torch.from_numpy(sx).cuda(), torch.from_numpy(sw).cuda()
    acc = (cr.convrot_w4a4_gemm_i32 if bits == 4 else cr.convrot_w8a8_gemm_i32)(Xq, Wq, M, N, K)
    y, yb = (gemm(Xq, scales[0], Wq, scales[1], K, bias=b) for b in (None, bias))
    torch.cuda.synchronize()
    t = torch.from_numpy(qx).cuda().double() @ torch.from_numpy(qw).cuda().double().T      # whole numbers below 2^53: exact in doubles
    ref = t.round().int()
    assert torch.equal(acc, ref)
    rows = np.unique(np.concatenate([np.arange(0, M, 53), [M - 1]]))
    d = bf16_ulp_diff(bf16_to_host_bits(y[torch.from_numpy(rows).cuda()]), oracle.dequant(ref.cpu().numpy()[rows], sx[rows], sw))
    assert d.max() <= 1
    # one rounding to bf16 (2^-8 of the value at most) of a value that took three fp32 roundings of the product and its sum with the bias
    t *= scales[0].double()[:, None] * scales[1].double()
    full = t + bias.double()
    assert ((yb.double() - full).abs() <= full.abs() * (2.0 ** -8 * (1 + 2.0 ** -20)) + (t.abs() + full.abs()) * 2.0 ** -22).all()
