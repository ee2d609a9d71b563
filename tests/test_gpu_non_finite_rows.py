"""A NaN or an infinity in a row of X or W leaves every other row as it would be without it (include/convrot.h): codes and scales of
rotate+quantise in each split of a row, of few rows and of many, outputs of the one-launch forwards and of the two-launch one, bit for bit."""
import pytest
import torch

from gpu_util import forward_rules, two_launches

INF, NAN = float("inf"), float("nan")
GROUPS = (4, 16, 64, 256, 1024)


def spoil(x):
    """x with non-finite elements in a middle row and, of more than three, the first and the last one, at the ends of the row and inside;
    the rows that stay."""
    bad, M = x.clone(), x.shape[0]
    keep = torch.ones(M, dtype=torch.bool, device=x.device)
    bad[M // 2, -1] = NAN
    bad[M // 2, x.shape[1] // 2] = -INF
    keep[M // 2] = False
    if M > 3:
        bad[0, 0] = INF
        bad[M - 1, -1] = -INF
        bad[M - 1, 5] = INF
        keep[[0, M - 1]] = False
    return bad, keep


def same_rows(a, b, keep, bits):
    """Whether two code matrices agree in the rows to keep.  4 bits: blocks of 32 rows, 64 bytes of each and then 32 of each; 8 bits: panels
    of 16 rows, 64 bytes of each.  Bytes past the last row count as kept."""
    n = torch.arange(3072 if bits == 4 else 1024, device=a.device)
    row = torch.where(n < 2048, n // 64, (n - 2048) // 32)
    rows = 32 if bits == 4 else 16
    groups = -(-keep.numel() // rows)
    k = torch.ones(groups * rows, dtype=torch.bool, device=a.device)
    k[:keep.numel()] = keep
    differ = (a != b).view(groups, -1, n.numel())
    return not (differ & k.view(groups, 1, rows)[:, :, row]).any()


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("K", (256, 512, 1024, 2048, 3072, 4096, 5120, 8192, 12288, 16384, 20480, 40960))
def test_rotquant(K, bits):
    from paper_2512_03673_amd import binding as cr
    size, rotquant = (cr.packed_bytes, cr.convrot_rotquant_act) if bits == 4 else (cr.packed_bytes8, cr.convrot_rotquant_act8)
    M = 67 if K <= 4096 else 9
    x = torch.randn(M, K, generator=torch.Generator(device="cuda").manual_seed(K + bits), device="cuda").to(torch.bfloat16)
    bad, keep = spoil(x)
    for g in GROUPS:
        if K % g:
            continue
        print(f"bits={bits} M={M} K={K} g={g}", flush=True)
        q, s = zip(*(rotquant(v, g, Xq=torch.full((size(M, K),), 0x5A, dtype=torch.uint8, device="cuda")) for v in (x, bad)))
        torch.cuda.synchronize()
        assert torch.equal(s[0][keep], s[1][keep]) and same_rows(q[0], q[1], keep, bits), g


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("K", (1280, 2048, 3072, 4096, 5120, 8192, 12288))
def test_rotquant_of_many_rows(K, bits):
    """Past the lines up to which a row is a block of its own (csrc/rotquant_kernel.h): two rows side by side in a wavefront up to K = 4096, in units
    and (4 bits, from some 2e7 elements on) in whole chunks, single rows of whole chunks beyond.  The first and the last row, each of another half
    of its pair, are spoiled."""
    from paper_2512_03673_amd import binding as cr
    size, rotquant = (cr.packed_bytes, cr.convrot_rotquant_act) if bits == 4 else (cr.packed_bytes8, cr.convrot_rotquant_act8)
    for M in [12 * 256 // -(-K // 1024) + 1] + ([-(-20_000_000 // K), -(-34_000_000 // K)] if bits == 4 and K <= 4096 else []):
        M += M % 2
        x = torch.randn(M, K, generator=torch.Generator(device="cuda").manual_seed(K + bits), device="cuda").to(torch.bfloat16)
        bad, keep = spoil(x)
        assert not keep[0] and keep[1] and keep[M - 2] and not keep[M - 1]
        for g in GROUPS:
            if K % g:
                continue
            print(f"bits={bits} M={M} K={K} g={g}", flush=True)
            q, s = zip(*(rotquant(v, g, Xq=torch.full((size(M, K),), 0x5A, dtype=torch.uint8, device="cuda")) for v in (x, bad)))
            torch.cuda.synchronize()
            assert torch.equal(s[0][keep], s[1][keep]) and same_rows(q[0], q[1], keep, bits), g


FORWARDS = [(3, 100, 1024), (8, 260, 1024), (4, 5000, 3072), (3, 300, 5120), (20, 200, 3072), (300, 390, 1024)]
TWO_LAUNCHES = [(20, 5000, 3072), (300, 1100, 2048), (1200, 500, 1024)]


def test_forwards_take_each_way():
    for bits in (4, 8):
        rules = forward_rules(FORWARDS)
        assert any(r["one"] for r in rules.values()) and any(r[f"row_tiles{bits}"] for r in rules.values())
        assert two_launches(TWO_LAUNCHES, bits) == TWO_LAUNCHES


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("M,N,K", FORWARDS + TWO_LAUNCHES)
def test_forward(M, N, K, bits):
    from paper_2512_03673_amd import binding as cr
    prepare, forward = (cr.convrot_prepare_weight, cr.convlinear4bit_forward) if bits == 4 else (cr.convrot_prepare_weight8, cr.convlinear8bit_forward)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K + bits)
    x, w = (torch.randn(r, K, generator=gen, device="cuda").to(torch.bfloat16) for r in (M, N))
    bad, keep = spoil(x)
    bad_w, keep_w = spoil(w)
    for g in GROUPS:
        print(f"bits={bits} M={M} N={N} K={K} g={g}", flush=True)
        y, yx, yw = (forward(a, *prepare(b, g), g) for a, b in ((x, w), (bad, w), (x, bad_w)))
        torch.cuda.synchronize()
        assert torch.isfinite(y).all()
        assert torch.equal(y[keep], yx[keep]) and torch.equal(y[:, keep_w], yw[:, keep_w]), g
