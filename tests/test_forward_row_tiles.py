"""The one-launch forward in tiles of rows against the two launches it stands for: same codes, scales and output, bit for bit, at the
edges of its tiles: rows that do not divide among them or among the code layouts' blocks of 16 and 32, one to four stretches of 1024
elements a row, each block width, ragged N and K.  Which shapes those are is a host function, asked on the CPU."""
import ctypes
import shutil
import subprocess

import pytest
import torch

import test_forward_small
from gpu_util import CSRC, forward_rules

# (M, N, K): (rows, columns) of a block
SHAPES = {(9, 64, 256): (9, 32), (17, 33, 32): (9, 32), (31, 1000, 96): (16, 32), (33, 500, 1024): (11, 32), (256, 1024, 1024): (16, 64), (250, 512, 320): (16, 32),
          (257, 960, 1024): (16, 64), (100, 1537, 1056): (8, 128), (389, 437, 1056): (8, 128), (40, 6100, 1024): (14, 128), (4096, 77, 1024): (16, 128),
          (25, 513, 2048): (7, 32), (13, 700, 2080): (5, 32), (6, 90, 4096): (3, 32), (3, 5000, 160): (3, 32), (16, 8192, 1280): (8, 64), (11, 8191, 1280): (6, 64)}
SHAPES8 = [s for s, (_, columns) in SHAPES.items() if s[2] * columns * 2 <= 144 * 1024]
OTHERS = [(4097, 64, 64), (256, 2049, 1024), (389, 437, 1312), (257, 1000, 2048), (60, 1024, 3072), (1, 32769, 32), (2, 64, 4128), (2 ** 31 - 1, 2 ** 31 - 1, 65536)]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_which_shapes_take_row_tiles(tmp_path):
    src = tmp_path / "rule.cpp"
    src.write_text('#include "gemm_plan.h"\n#include <cstdio>\n#include <cstdlib>\nusing namespace convrot::gemm;\nint main(int n, char **v) {\n'
                   '  for (int i = 1; i + 2 < n; i += 3) {\n    const long M = atol(v[i]), N = atol(v[i + 1]), K = atol(v[i + 2]);\n'
                   '    const bool four = forward_in_row_tiles(M, N, K, 4);\n    const RowTiles t = four ? forward_row_tiles(M, N, K) : RowTiles{0, 0};\n'
                   '    std::printf("%d %d %d %d\\n", four, forward_in_row_tiles(M, N, K, 8), t.rows, t.columns);\n  }\n}\n')
    exe = str(tmp_path / "rule")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", exe, str(src)], check=True)
    many = [(M, N, K) for M in (1, 2, 5, 15, 16, 17, 100, 255, 1000, 4096) for N in (1, 31, 32, 33, 64, 1000, 8192, 32768) for K in (32, 1024, 1056, 2048, 2080, 3104, 4096)]
    shapes = list(SHAPES) + OTHERS + many
    out = subprocess.run([exe] + [str(d) for s in shapes for d in s], check=True, capture_output=True, text=True).stdout.split()
    got = {s: tuple(int(o) for o in out[4 * i:4 * i + 4]) for i, s in enumerate(shapes)}
    for s, tile in SHAPES.items():
        assert got[s] == (1, int(s in SHAPES8), *tile), s
    for s in OTHERS:
        assert got[s][:2] == (0, 0), s
    for (M, N, K), (four, eight, rows, columns) in got.items():      # what the kernel is built for
        assert four or not eight
        if four:
            assert 1 <= rows <= 16 and rows * -(-K // 1024) <= 16 and columns in (32, 64, 128) and -(-M // rows) * -(-N // columns) <= 256


@pytest.mark.gpu
@pytest.mark.parametrize("bits,M,N,K", [(4, *s) for s in SHAPES] + [(8, *s) for s in SHAPES8])
def test_one_launch_equals_two(bits, M, N, K):
    test_forward_small.test_one_launch_equals_two(M, N, K, bits)


# a block's rows of at most six, or a few stretches; long rows in up to 160 blocks, of groups up to 256; and past that
IN_GRAPH = [(9, 9000, 160), (6, 90, 4096), (1, 32768, 1024), (17, 8192, 1024), (8, 9216, 1024), (20, 6000, 640), (8, 20000, 320)]
IN_GRAPH_TO_256 = [(25, 513, 1056), (160, 512, 1024), (77, 1024, 1024)]
NOT_IN_GRAPH = [(256, 1024, 1024), (389, 437, 1056), (250, 1000, 1152), (22, 4000, 640), (34, 8193, 320), (9, 22285, 128), (160, 513, 1024), (160, 512, 992)]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_which_shapes_take_row_tiles_in_a_graph():
    rules = forward_rules(IN_GRAPH + IN_GRAPH_TO_256 + NOT_IN_GRAPH)
    assert all(r["row_tiles4"] and not r["one"] for r in rules.values()), rules
    assert [s for s, r in rules.items() if r["in_graph"]] == IN_GRAPH + IN_GRAPH_TO_256 and [s for s, r in rules.items() if r["in_graph1024"]] == IN_GRAPH


def kernels_of(graph, library):
    """Nodes of a captured graph, all of which are kernels."""
    n, kind = ctypes.c_size_t(), ctypes.c_int()
    graph = ctypes.c_void_p(graph)
    assert library.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert library.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
    for node in nodes:
        assert library.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0 and kind.value == 0
    return n.value


@pytest.mark.gpu
@pytest.mark.parametrize("bits", (4, 8))
@pytest.mark.parametrize("M,N,K,g", [(8, 9216, 1024, 1024), (256, 1024, 1024, 16), (77, 1024, 1024, 256), (77, 1024, 1024, 1024)])
def test_captured_forward(M, N, K, g, bits):
    """A captured forward of row tiles records one kernel or two, by the rule, and gives the bytes of the call."""
    from paper_2512_03673_amd import binding as cr
    prepare, forward, space, size = ((cr.convrot_prepare_weight, cr.convlinear4bit_forward, cr.workspace_bytes, cr.packed_bytes) if bits == 4 else
                                     (cr.convrot_prepare_weight8, cr.convlinear8bit_forward, cr.workspace_bytes8, cr.packed_bytes8))
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    X, W = (torch.randn(r, K, generator=gen, device="cuda").to(torch.bfloat16) for r in (M, N))
    Wq, ws = prepare(W, g)
    Y, work = torch.empty(M, N, dtype=torch.bfloat16, device="cuda"), torch.zeros(space(M, K), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        forward(X, Wq, ws, g, Y, work)
    assert kernels_of(graph.raw_cuda_graph(), cr.load()) == (1 if (M, N, K) in IN_GRAPH or (g <= 256 and (M, N, K) in IN_GRAPH_TO_256) else 2)
    graph.instantiate()
    for rep in range(3):
        X.copy_(torch.randn(M, K, generator=gen, device="cuda") * (rep + 1))
        called = torch.zeros_like(work)
        y = forward(X, Wq, ws, g, workspace=called)
        Y.zero_()
        work.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        written = size(M, K) + 4 * M
        assert torch.equal(Y, y) and torch.equal(work[:written], called[:written]), rep
