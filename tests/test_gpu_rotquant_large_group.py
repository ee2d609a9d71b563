"""Groups of 1024 in rows whose wavefront count is no power of two, or whose last wavefront is partly idle: the top digit of
the rotation runs over a lane's four units there, in blocks as long as the row."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_codes, to_dev_bf16, ulp_diff_f32, unpack_host, unpack_host8
from paper_2512_03673_amd import workloads as wl


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("M,K", [(1, 3072), (45, 3072), (33, 4096), (35, 5120), (31, 11264), (3, 17408), (34, 20480), (2, 33792), (1, 64512)])
def test_rows_of_any_number_of_groups(M, K, bits):
    from paper_2512_03673_amd import binding as cr
    spec = wl.LayerSpec(f"lg_{M}_{K}", M=M, K=K, N=8, group=1024, x_col_count=K // 100, x_row_count=1, seed=17)
    x = wl.make_activation(spec)
    q, s = (cr.convrot_rotquant_act if bits == 4 else cr.convrot_rotquant_act8)(to_dev_bf16(x), 1024)
    torch.cuda.synchronize()
    qo, so = oracle.rotquant(x, 1024, qmax=7 if bits == 4 else 127)
    if bits == 4:
        check_codes(unpack_host(q, M, K), s.cpu().numpy(), qo, so, f"M={M} K={K}")
    else:
        d = np.abs(unpack_host8(q, M, K).astype(np.int16) - qo)
        assert d.max() <= 1 and (d == 0).mean() >= 0.9999
        assert ulp_diff_f32(s.cpu().numpy(), so).max() <= 2
