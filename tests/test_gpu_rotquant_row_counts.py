"""How a row is split over lanes and wavefronts depends on the number of rows too (few rows, many, very many): every split gives
the codes, scales and zero padding of the few-row one, byte for byte, which test_gpu_rotquant_splits.py compares with the oracle.  Row
counts are the first past each line of the choice (12 wavefronts of 1024 elements a compute unit; at 4 bits 2e7 elements, or 3.4e7 of
groups up to 16 in rows of up to 1536 or of more than 3072)."""
import pytest
import torch

LENGTHS = (1056, 2048, 2080, 3072, 3104, 4096, 4128, 6144, 6176, 10240, 12288, 12320)


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("K", LENGTHS)
def test_row_counts(K, bits):
    from paper_2512_03673_amd import binding as cr
    size, rotquant = (cr.packed_bytes, cr.convrot_rotquant_act) if bits == 4 else (cr.packed_bytes8, cr.convrot_rotquant_act8)
    group_rows = 32 if bits == 4 else 16
    gen = torch.Generator(device="cuda").manual_seed(K)
    for g in (4, 16, 64, 256, 1024):
        k = -(-K // max(g, 32)) * max(g, 32)
        few = 12 * 256 // -(-k // 1024)
        lines = [20_000_000] + ([34_000_000] if bits == 4 and g == 16 and (k <= 1536 or k > 3072) else [])
        for M in [few, few + 1] + ([-(-n // k) - less for n in lines for less in (1, 0)] if k <= 4096 and g in (16, 256, 1024) else []):
            print(f"bits={bits} M={M} K={k} g={g}", flush=True)
            x = torch.randn(M, k, generator=gen, device="cuda")
            x[:, ::97] *= 30.0
            x[M // 2] = 0.0
            x = x.to(torch.bfloat16)
            q = torch.full((size(M, k) + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
            s = torch.full((M + 64,), 3.0, device="cuda")
            rotquant(x, g, Xq=q[:size(M, k)], x_scale=s[:M])
            assert (q[size(M, k):] == 0x5A).all() and (s[M:] == 3.0).all()
            slab = max(1, min(few, 512) // group_rows) * group_rows
            for r in range(0, M, slab):
                n = min(slab, M - r)
                part = torch.full((size(n, k),), 0x5A, dtype=torch.uint8, device="cuda")
                part, ps = rotquant(x[r:r + n], g, Xq=part)
                assert torch.equal(part, q[size(r, k):size(r, k) + size(n, k)]) and torch.equal(ps, s[r:r + n]), r
