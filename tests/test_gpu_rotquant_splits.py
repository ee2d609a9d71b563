"""Rotate+quantise at the edges of its splits of a row over lanes and wavefronts: the shortest and the longest row of each, rows
that end inside a column of 64 elements or inside a stage of the code layout, row counts around a block's.  Codes, scales and
zero padding against the oracle; bytes behind the matrix and scales behind the last row stay as they were."""
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
