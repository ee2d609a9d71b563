"""The tiles that take a ring of four stages in a launch of one round (csrc/gemm_plan.h: deep_ring): both rings of both, from 16 stages on (of
128 codes at 4 bits, of 64 at 8) in up to 256 tiles, and else; whole and ragged edges, the last stage padded, with and without a bias.
Which ring a shape takes is asked on the CPU.  Accumulators bit for bit against the exact integer product of the same codes, outputs
against it dequantised."""
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle
from gpu_util import CSRC, bf16_to_host_bits, bf16_ulp_diff, codes4_to_dev, codes8_to_dev, gemm_plans

# bits, M, N, K, ring of four.  (At 4 bits the plan takes 192 x 192 tiles of one round with a few stages or with 16 and more.)
SHAPES = [(4, 3000, 2900, 2048, True), (4, 2881, 3072, 1952, True), (4, 3070, 2876, 2080, True), (4, 2944, 3001, 3072, True), (4, 3072, 3072, 3072, True),
          (4, 3001, 3070, 160, False), (4, 3072, 3072, 128, False), (4, 1621, 9459, 2592, False),
          (8, 511, 12280, 1024, True), (8, 511, 12285, 960, False), (8, 509, 12285, 1120, True), (8, 512, 12281, 3040, True), (8, 512, 12288, 1024, True),
          (8, 512, 12288, 960, False), (8, 811, 10588, 1408, False)]


def rings(tmp_path):
    """(tiles, stages, ring of four) of each of SHAPES, by the expressions of the launchers"""
    src, exe = tmp_path / "ring.cpp", str(tmp_path / "ring")
    src.write_text('#include "gemm_plan.h"\n#include <cstdio>\nusing namespace convrot::gemm;\nint main() {\n  long b, M, N, K;\n'
                   '  while (std::scanf("%ld %ld %ld %ld", &b, &M, &N, &K) == 4) {\n'
                   '    const long tiles = b == 4 ? tiles_of(M, N, 192, 192) : tiles_of(M, N, 128, 192), stages = b == 4 ? (K + 127) / 128 : (K + 63) / 64;\n'
                   '    std::printf("%ld %ld %d\\n", tiles, stages, (int)deep_ring(tiles, stages));\n  }\n}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(src)], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, input="\n".join(" ".join(map(str, s[:4])) for s in SHAPES)).stdout.split()
    return [tuple(int(v) for v in out[3 * i:3 * i + 3]) for i in range(len(SHAPES))]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_shapes_lie_on_both_sides_of_the_line(tmp_path):
    plans = gemm_plans([s[1:4] for s in SHAPES])
    got = rings(tmp_path)
    for (bits, M, N, K, deep), ring in zip(SHAPES, got):
        assert plans[(M, N, K)][bits == 8] == ("192x192" if bits == 4 else "128x192") and ring[2] == deep, (bits, M, N, K, ring)
    for bits in (4, 8):
        mine = [r for s, r in zip(SHAPES, got) if s[0] == bits]
        assert any(t <= 256 and n == 16 for t, n, _ in mine) and any(t <= 256 and n < 16 for t, n, _ in mine) and any(t > 256 and n >= 16 for t, n, _ in mine)
    assert any(n == 15 for s, (t, n, _) in zip(SHAPES, got) if s[0] == 8)


@pytest.mark.gpu
@pytest.mark.parametrize("bits,M,N,K", [s[:4] for s in SHAPES])
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
    bias = rng.standard_normal(N).astype(np.float32) * 50
    bias = torch.from_numpy(bias).cuda().to(torch.bfloat16)
    gemm = cr.convrot_w4a4_gemm_dequant if bits == 4 else cr.convrot_w8a8_gemm_dequant
    scales = torch.from_numpy(sx).cuda(), torch.from_numpy(sw).cuda()
    acc = (cr.convrot_w4a4_gemm_i32 if bits == 4 else cr.convrot_w8a8_gemm_i32)(Xq, Wq, M, N, K)
    y, yb = (gemm(Xq, scales[0], Wq, scales[1], K, bias=b) for b in (None, bias))
    torch.cuda.synchronize()
    # whole numbers below 2^53: the product in doubles is exact
    t = torch.from_numpy(qx).cuda().double() @ torch.from_numpy(qw).cuda().double().T
    ref = t.round().int()
    assert torch.equal(acc, ref)
    rows = np.unique(np.concatenate([np.arange(0, M, 97), [M - 1]]))
    d = bf16_ulp_diff(bf16_to_host_bits(y[torch.from_numpy(rows).cuda()]), oracle.dequant(ref.cpu().numpy()[rows], sx[rows], sw))
    assert d.max() <= 1
    # one rounding to bf16 (2^-8 of the value at most) of a value that took three fp32 roundings of the product and its sum with the bias
    t *= scales[0].double()[:, None] * scales[1].double()
    full = t + bias.double()
    assert ((yb.double() - full).abs() <= full.abs() * (2.0 ** -8 * (1 + 2.0 ** -20)) + (t.abs() + full.abs()) * 2.0 ** -22).all()
