"""GPU: the library launches on the stream it is given, calls on different streams do not disturb each other,
and a forward can be captured into a HIP graph and replayed (it allocates nothing and records no memset).

The expected outputs are the library's own results on the default stream, which the parity tests hold
against the oracle; one case here is checked against the oracle directly as well.
"""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import oracle
from gpu_util import bf16_to_host_bits, check_output, gemm_plans, to_dev_bf16, two_launches
from paper_2512_03673_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cr():
    from paper_2512_03673_amd import binding
    binding.load()
    return binding


def layer(M, K, N, g, seed):
    spec = wl.LayerSpec(f"stream_{seed}", M=M, K=K, N=N, group=g, seed=seed)
    x, w = wl.make_layer(spec)
    return spec, x, w


# a forward of one launch as it is called, and one of two whatever the code width
ONE, TWO = (300, 1024, 520), (1200, 1024, 1000)


def test_one_and_two_launches():
    shapes = [(M, N, K) for M, K, N in (ONE, TWO)]
    assert two_launches(shapes, 4) == two_launches(shapes, 8) == shapes[1:]


@pytest.mark.parametrize("M,K,N", (ONE, TWO))
def test_forward_runs_on_the_given_stream(cr, M, K, N):
    # X is produced on a side stream by a long chain of kernels; the forward is queued behind it on the same
    # stream.  Launched anywhere else it would read X before the chain has written it (torch's side streams
    # do not synchronise with the default stream).
    spec, x, w = layer(M, K, N, 16, 11)
    X = to_dev_bf16(x)
    wq, ws = cr.convrot_prepare_weight(to_dev_bf16(w), 16)
    y_ref = cr.convlinear4bit_forward(X, wq, ws, 16)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    Xs = torch.zeros_like(X)
    big = torch.ones((8192, 8192), device="cuda")
    Y = torch.zeros_like(y_ref)
    wsb = torch.empty((cr.workspace_bytes(spec.M, spec.K),), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(20):
            big = big * 1.0001 + 0.5          # milliseconds of work ahead of the copy
        Xs.copy_(X)
        cr.convlinear4bit_forward(Xs, wq, ws, 16, Y, wsb, stream=side)
    side.synchronize()
    assert torch.equal(Y, y_ref)
    (qx, sx), (qw, sw) = oracle.rotquant(x, 16), oracle.rotquant(w, 16)
    yo = oracle.dequant(oracle.int_gemm(qx, qw), sx, sw)
    check_output(bf16_to_host_bits(Y), yo, "forward on a side stream")


def test_calls_on_two_streams_do_not_disturb_each_other(cr):
    # two layers whose GEMMs take different tiles, each with its own buffers, queued alternately on two streams
    cases = []
    for M, K, N, g, seed in ((3072, 256, 3072, 16, 21), (700, 2048, 900, 64, 22)):
        spec, x, w = layer(M, K, N, g, seed)
        X = to_dev_bf16(x)
        wq, ws = cr.convrot_prepare_weight(to_dev_bf16(w), g)
        y_ref = cr.convlinear4bit_forward(X, wq, ws, g)
        Y = torch.empty_like(y_ref)
        wsb = torch.empty((cr.workspace_bytes(M, K),), dtype=torch.uint8, device="cuda")
        cases.append((X, wq, ws, g, Y, wsb, y_ref, torch.cuda.Stream()))
    assert {p4 for p4, _ in gemm_plans([(3072, 3072, 256), (700, 900, 2048)]).values()} == {"192x192", "64x64"}
    torch.cuda.synchronize()
    for rep in range(10):
        for X, wq, ws, g, Y, wsb, y_ref, s in cases:
            with torch.cuda.stream(s):
                if rep == 9:
                    Y.zero_()
                cr.convlinear4bit_forward(X, wq, ws, g, Y, wsb, stream=s)
    torch.cuda.synchronize()
    for X, wq, ws, g, Y, wsb, y_ref, s in cases:
        assert torch.equal(Y, y_ref)


@pytest.mark.parametrize("M,K,N", ((520, 1024, 300), TWO))
@pytest.mark.parametrize("bits", (4, 8))
def test_forward_in_a_hip_graph(cr, bits, M, K, N):
    spec, x, w = layer(M, K, N, 16, 31 + bits)
    prep, fwd, wsbytes = ((cr.convrot_prepare_weight, cr.convlinear4bit_forward, cr.workspace_bytes) if bits == 4 else
                          (cr.convrot_prepare_weight8, cr.convlinear8bit_forward, cr.workspace_bytes8))
    X = to_dev_bf16(x)
    wq, ws = prep(to_dev_bf16(w), 16)
    bias = to_dev_bf16(wl.make_bias(spec))
    Y = torch.zeros((spec.M, spec.N), dtype=torch.bfloat16, device="cuda")
    wsb = torch.empty((wsbytes(spec.M, spec.K),), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fwd(X, wq, ws, 16, Y, wsb, bias=bias)
    torch.cuda.synchronize()
    rng = np.random.default_rng(5)
    for rep in range(4):
        # new input in the captured buffer, eager work and a synchronisation between the replays
        x2 = wl.f32_to_bf16_bits((rng.standard_normal((spec.M, spec.K)) * (rep + 1)).astype(np.float32))
        X.copy_(to_dev_bf16(x2))
        y_eager = fwd(X, wq, ws, 16, bias=bias).clone()
        Y.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, y_eager), f"replay {rep}"


_FIRST_CALL_CAPTURED = r"""
import sys
import torch
sys.path.insert(0, sys.argv[1])
from paper_2512_03673_amd import binding as cr
bits = int(sys.argv[2])
fwd, packed, wsbytes = ((cr.convlinear4bit_forward, cr.packed_bytes, cr.workspace_bytes) if bits == 4 else
                        (cr.convlinear8bit_forward, cr.packed_bytes8, cr.workspace_bytes8))
M, K, N, g = 520, 1024, 3000, 16
torch.manual_seed(3)
X = torch.randn((M, K), device="cuda").to(torch.bfloat16)
# any bytes are a valid code matrix (every six-bit pattern is a finite E2M3 number, every byte an int8 code), so the
# weight needs no library call; the K padding must hold zero codes, and K = 1024 has none
wq = torch.randint(0, 256, (packed(N, K),), dtype=torch.uint8, device="cuda")
ws = torch.rand((N,), device="cuda") * 1e-3 + 1e-4
bias = torch.randn((N,), device="cuda").to(torch.bfloat16)
Y = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
wsb = torch.empty((wsbytes(M, K),), dtype=torch.uint8, device="cuda")
torch.cuda.synchronize()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph):                       # the first call into the library in this process
    fwd(X, wq, ws, g, Y, wsb, bias=bias)
for rep in range(3):
    X.copy_(torch.randn((M, K), device="cuda").to(torch.bfloat16) * (rep + 1))
    Y.zero_()
    torch.cuda.synchronize()
    graph.replay()
    torch.cuda.synchronize()
    y_eager = fwd(X, wq, ws, g, bias=bias)
    torch.cuda.synchronize()
    assert torch.isfinite(Y.float()).all() and Y.float().abs().max() > 0
    assert torch.equal(Y, y_eager), f"replay {rep}"
print("first call captured: ok")
"""


@pytest.mark.parametrize("bits", (4, 8))
def test_first_library_call_of_a_process_under_capture(bits):
    # The library keeps no set-up for a first eager call to do: a process whose very first call into it is made
    # under stream capture gets a working graph.  Run in a child process, which has not touched the library.
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", _FIRST_CALL_CAPTURED, root, str(bits)], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0 and "first call captured: ok" in r.stdout, r.stdout + r.stderr


def _stream_of_memory(t):
    """The stream whose memory torch's allocator took the tensor from."""
    found = [s["stream"] for s in torch.cuda.memory_snapshot() if s["address"] <= t.data_ptr() < s["address"] + s["total_size"]]
    assert len(found) == 1
    return found[0]


def test_new_tensors_belong_to_the_stream_of_the_call(cr):
    spec, x, w = layer(1200, 1024, 1000, 16, 41)
    M, K, N, g = spec.M, spec.K, spec.N, 16
    X, W, side = to_dev_bf16(x), to_dev_bf16(w), torch.cuda.Stream()
    Xq, xs = cr.convrot_rotquant_act(X, g)
    Wq, ws = cr.convrot_prepare_weight(W, g)
    Xq8, xs8 = cr.convrot_rotquant_act8(X, g)
    Wq8, ws8 = cr.convrot_prepare_weight8(W, g)
    calls = [lambda s: cr.convrot_prepare_weight(W, g, stream=s), lambda s: cr.convrot_rotquant_act8(X, g, stream=s),
             lambda s: cr.convrot_w4a4_gemm_dequant(Xq, xs, Wq, ws, K, stream=s), lambda s: cr.convrot_w8a8_gemm_dequant(Xq8, xs8, Wq8, ws8, K, stream=s),
             lambda s: cr.convlinear4bit_forward(X, Wq, ws, g, stream=s), lambda s: cr.convlinear8bit_forward(X, Wq8, ws8, g, stream=s),
             lambda s: cr.convrot_w4a4_gemm_i32(Xq, Wq, M, N, K, stream=s), lambda s: cr.convrot_w8a8_gemm_i32(Xq8, Wq8, M, N, K, stream=s),
             lambda s: cr.convrot_unpack_codes(Xq, M, K, stream=s), lambda s: cr.convrot_rotated_absmax(X, g, 1, stream=s)]
    torch.cuda.synchronize()
    for i, call in enumerate(calls):
        ref = call(None)
        ref = ref if isinstance(ref, tuple) else (ref,)
        torch.cuda.synchronize()
        for stream in (side, torch.cuda.ExternalStream(side.cuda_stream), torch.cuda.current_stream()):
            got = call(stream)
            assert torch.cuda.current_stream() == torch.cuda.default_stream()
            torch.cuda.synchronize()
            for a, b in zip(got if isinstance(got, tuple) else (got,), ref):
                assert _stream_of_memory(a) == stream.cuda_stream, (i, stream)
                assert a.dtype == torch.uint8 or torch.equal(a, b)       # (a code matrix has bytes past its rows that nobody writes)
        with torch.cuda.stream(side):
            got = call(torch.cuda.default_stream())
        torch.cuda.synchronize()
        assert all(_stream_of_memory(t) == 0 for t in (got if isinstance(got, tuple) else (got,))), i


@pytest.mark.parametrize("bits", (4, 8))
def test_forward_without_buffers_on_another_stream(cr, bits):
    # The side stream is held up, so that the call's kernels run after everything that the current stream is given next: new
    # tensors of the sizes that the call made and gave back, written all over.  Then the current stream is held up while it reads an
    # output that is given back, and the side stream runs on with new calls.
    prep, fwd, wsbytes = ((cr.convrot_prepare_weight, cr.convlinear4bit_forward, cr.workspace_bytes) if bits == 4 else
                          (cr.convrot_prepare_weight8, cr.convlinear8bit_forward, cr.workspace_bytes8))
    spec, x, w = layer(1200, 1024, 1000, 16, 43)
    X, side = to_dev_bf16(x), torch.cuda.Stream()
    wq, ws = prep(to_dev_bf16(w), 16)
    y_ref = fwd(X, wq, ws, 16).clone()
    X2 = torch.full_like(X, 2.0)
    torch.cuda.synchronize()
    for _ in range(3):
        with torch.cuda.stream(side):
            torch.cuda._sleep(20_000_000)
        y = fwd(X, wq, ws, 16, stream=side)
        junk = [torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda") for n in 4 * [wsbytes(spec.M, spec.K), 2 * spec.M * spec.N]]
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda._sleep(20_000_000)
        seen = y + 0
        del y, junk
        for _ in range(4):
            fwd(X2, wq, ws, 16, stream=side)
        torch.cuda.synchronize()
        assert torch.equal(seen, y_ref)
