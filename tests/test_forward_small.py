"""The one-launch forward of a few rows against the two launches it stands for (rotate+quantise, then GEMM): same codes and
scales in the workspace, same output, bit for bit, at the edges of what it takes: one row, as many rows and as long rows as
it allows, padded K, ragged N, every group."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle
from gpu_util import bf16_to_host_bits, check_output, to_dev_bf16, two_launches
from paper_2512_03673_amd import workloads as wl

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_03673_amd", "csrc")
SHAPES = [(1, 1, 32), (8, 1024, 1024), (1, 33, 96), (3, 77, 160), (8, 300, 1024), (8, 4097, 672), (7, 257, 256), (2, 4096, 4096), (4, 4096, 4096),
          (1, 4095, 16384), (1, 9216, 3072), (4, 16384, 64), (3, 1000, 5120), (5, 8192, 1024), (1, 8192, 15360)]
# past that one launch: in tiles of rows, mostly (test_forward_row_tiles.py), and in two launches
NOT_SO = [(9, 64, 256), (8, 16384, 64), (1, 16385, 64), (5, 64, 4096), (1, 64, 17408), (1, 8193, 15360), (64, 3072, 3072), (0, 64, 64)]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_which_shapes_take_one_launch(tmp_path):
    src = tmp_path / "rule.cpp"
    src.write_text('#include "gemm_plan.h"\n#include <cstdio>\n#include <cstdlib>\nint main(int n, char **v) {\n  for (int i = 1; i + 2 < n; i += 3)\n'
                   '    std::printf("%d\\n", (int)convrot::gemm::forward_in_one(atol(v[i]), atol(v[i + 1]), atol(v[i + 2])));\n}\n')
    exe = str(tmp_path / "rule")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(src)], check=True)
    shapes = SHAPES + NOT_SO[:-1] + [(2 ** 31 - 1, 2 ** 31 - 1, 65536)]
    out = subprocess.run([exe] + [str(d) for s in shapes for d in s], check=True, capture_output=True, text=True).stdout.split()
    assert [int(o) for o in out] == [int(s in SHAPES) for s in shapes]
    two = [(1, 64, 17408), (1, 8193, 15360), (64, 3072, 3072)]
    assert two_launches(NOT_SO[:-1], 4) == two and two_launches(NOT_SO[:-1], 8) == [(5, 64, 4096)] + two


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("M,N,K", SHAPES + NOT_SO[:2] + [(1, 64, 17408), (64, 3072, 3072)])
def test_one_launch_equals_two(M, N, K, bits):
    from paper_2512_03673_amd import binding as cr
    eight = "8" if bits == 8 else ""
    prepare, rotquant = getattr(cr, "convrot_prepare_weight" + eight), getattr(cr, "convrot_rotquant_act" + eight)
    gemm = cr.convrot_w8a8_gemm_dequant if bits == 8 else cr.convrot_w4a4_gemm_dequant
    forward = cr.convlinear8bit_forward if bits == 8 else cr.convlinear4bit_forward
    size, space = getattr(cr, "packed_bytes" + eight)(M, K), getattr(cr, "workspace_bytes" + eight)(M, K)
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    x = wl.f32_to_bf16_bits((rng.standard_normal((M, K)) * np.exp(rng.uniform(-2, 2, (1, K)))).astype(np.float32))
    w = wl.f32_to_bf16_bits((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
    bias = wl.f32_to_bf16_bits((rng.standard_normal(N) * 0.1).astype(np.float32))
    X, W, B = to_dev_bf16(x), to_dev_bf16(w), to_dev_bf16(bias)
    for g in (4, 16, 64, 256, 1024):
        if K % g:
            continue
        Wq, ws = prepare(W, g)
        Xq, xs = rotquant(X, g, Xq=torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda"))
        for b in (None, B):
            ref = gemm(Xq, xs, Wq, ws, K, bias=b)
            workspace = torch.full((space + 64,), 0x5A, dtype=torch.uint8, device="cuda")
            y = torch.full((M + 1, N), 3.0, dtype=torch.bfloat16, device="cuda")
            forward(X, Wq, ws, g, workspace=workspace[:space], bias=b, Y=y[:M])
            torch.cuda.synchronize()
            assert torch.equal(y[:M], ref) and (y[M] == 3.0).all(), g
            assert torch.equal(workspace[:size], Xq) and torch.equal(workspace[size:size + 4 * M].view(torch.float32), xs), g
            assert (workspace[size + 4 * M:] == 0x5A).all(), g
        if N == K:          # in place: the two launches read all of X before Y is written, and so does a forward laid over its input
            inout = X.clone()
            forward(inout, Wq, ws, g, Y=inout)
            torch.cuda.synchronize()
            assert torch.equal(inout, gemm(Xq, xs, Wq, ws, K)), g
    g = 16 if K % 16 == 0 else 4
    if N * K <= 2 ** 22 and bits == 4:
        Wq, ws = prepare(W, g)
        y = forward(X, Wq, ws, g)
        torch.cuda.synchronize()
        check_output(bf16_to_host_bits(y), oracle.convlinear4bit(x, w, g), f"{M} {N} {K}")
