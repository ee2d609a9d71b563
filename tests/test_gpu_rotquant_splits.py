"""Rotate+quantise at the edges of its splits of a row over lanes and wavefronts: the shortest and the longest row of each, rows
that end inside a column of 64 elements or inside a stage of the code layout, row counts around a block's.  Codes, scales and
zero padding against the oracle; bytes behind the matrix and scales behind the last row stay as they were.  The splits of many rows,
which rows of 1025 to 12288 elements have besides, on a wide spread of exponents."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_codes, to_dev_bf16, ulp_diff_f32, unpack_host, unpack_host8
from paper_2512_03673_amd import workloads as wl

LENGTHS = (32, 96, 256, 288, 512, 544, 1024, 1056, 2048, 2080, 3072, 3104, 4096, 4128, 6144, 6176, 10240, 12320, 16384, 16416, 32768, 32800, 65536)


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("K", LENGTHS)
def test_edges_of_the_splits(K, bits):
    from paper_2512_03673_amd import binding as cr
    size, rotquant = (cr.packed_bytes, cr.convrot_rotquant_act) if bits == 4 else (cr.packed_bytes8, cr.convrot_rotquant_act8)
    for g in (4, 16, 64, 256, 1024):
        k = -(-K // max(g, 32)) * max(g, 32)          # the next length that the group allows
        if k > 65536:
            continue
        for M in (1, 3, 33) if K <= 4128 else (2,):
            print(f"bits={bits} M={M} K={k} g={g}", flush=True)
            spec = wl.LayerSpec(f"sp_{M}_{k}", M=M, K=k, N=8, group=g, x_col_count=max(1, k // 100), x_row_count=1, seed=k + M)
            x = wl.make_activation(spec)
            buf = torch.full((size(M, k) + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
            scale = torch.full((M + 64,), 3.0, device="cuda")
            rotquant(to_dev_bf16(x), g, Xq=buf[:size(M, k)], x_scale=scale[:M])
            torch.cuda.synchronize()
            assert (buf[size(M, k):] == 0x5A).all() and (scale[M:] == 3.0).all()
            qo, so = oracle.rotquant(x, g, qmax=7 if bits == 4 else 127)
            s = scale[:M].cpu().numpy()
            if bits == 4:
                check_codes(unpack_host(buf[:size(M, k)], M, k), s, qo, so, f"M={M} K={k} g={g}")
            else:
                d = np.abs(unpack_host8(buf[:size(M, k)], M, k).astype(np.int16) - qo)
                assert d.max() <= 1 and (d == 0).mean() >= 0.9999
                assert ulp_diff_f32(s, so).max() <= 2


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("K", (1056, 2048, 3104, 4096, 6176, 10240, 12288))
def test_splits_of_many_rows(K, bits):
    """Past the lines of csrc/rotquant_kernel.h (launch_g): 12 wavefronts of 1024 elements a compute unit; at 4 bits 2e7 and 3.4e7 elements.  Rows of
    scales from 2^-60 to 2^60, columns e^-4 to e^4 apart; the first rows, the last ones and some between against the oracle."""
    from paper_2512_03673_amd import binding as cr
    size, rotquant = (cr.packed_bytes, cr.convrot_rotquant_act) if bits == 4 else (cr.packed_bytes8, cr.convrot_rotquant_act8)
    for g in (4, 16, 64, 256, 1024):
        k = -(-K // max(g, 32)) * max(g, 32)
        for M in [12 * 256 // -(-k // 1024) + 1] + ([-(-20_000_000 // k), -(-34_000_000 // k)] if bits == 4 and k <= 4096 else []):
            print(f"bits={bits} M={M} K={k} g={g}", flush=True)
            gen = torch.Generator(device="cuda").manual_seed(k + M + g)
            x = torch.randn(M, k, generator=gen, device="cuda")
            x *= torch.exp(torch.rand(k, generator=gen, device="cuda") * 8 - 4)
            x *= torch.exp2(torch.randint(-60, 61, (M, 1), generator=gen, device="cuda").float())
            x = x.to(torch.bfloat16)
            q, s = rotquant(x, g)
            torch.cuda.synchronize()
            step = 32 if bits == 4 else 16                       # rows of an output block
            group, parts = size(step, k), []
            for first in sorted({0, M // 2 // step * step, (M - 1) // step * step}):
                n = min(step, M - first)
                qo, so = oracle.rotquant(x[first:first + n].view(torch.int16).cpu().numpy().view(np.uint16), g, qmax=7 if bits == 4 else 127)
                codes = q[first // step * group:first // step * group + group]
                parts.append(((unpack_host if bits == 4 else unpack_host8)(codes, n, k), s[first:first + n].cpu().numpy(), qo, so))
            # All rows at once: a code whose quotient is within the rotation's fp32 rounding (some 1e-7 of the row's largest) of a tie may fall the other
            # way, about one in a million, and one would be more than 0.01 % of a last block that is a single row.
            codes, scale, qo, so = (np.concatenate(p) for p in zip(*parts))
            if bits == 4:
                check_codes(codes, scale, qo, so, f"M={M} K={k} g={g}")
            else:
                d = np.abs(codes.astype(np.int16) - qo)
                assert d.max() <= 1 and (d == 0).mean() >= 0.9999
                assert ulp_diff_f32(scale, so).max() <= 2
