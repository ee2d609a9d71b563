"""The extension module behind the per-layer calls of binding.py: what it rejects before anything is launched."""
import os
import shutil
import subprocess
import sys

import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from torch.utils._python_dispatch import TorchDispatchMode


@pytest.fixture(scope="module")
def cr():
    from paper_2512_03673_amd import binding, build
    if not (os.path.exists(build.LIB) and os.path.exists(build.CALLS)):
        build.build(verbose=False)
    return binding


def test_rejects_what_is_no_gpu_tensor(cr):
    x, s = torch.zeros(4, 32, dtype=torch.bfloat16), torch.zeros(4)
    q = torch.zeros(4096, dtype=torch.uint8)
    for f, args, name in ((cr.convlinear4bit_forward, (x, q, s, 16), "X"), (cr.convlinear8bit_forward, (x, q, s, 16), "X"),
                          (cr.convlinear4bit_forward_noalloc, (x, q, s, 16, x), "X"), (cr.convrot_prepare_weight, (x, 16), "W"),
                          (cr.convrot_rotquant_act, (x, 16), "X"), (cr.convrot_prepare_weight8, (x, 16), "W"),
                          (cr.convrot_w4a4_gemm_dequant, (q, s, q, s, 32), "x_scale"), (cr.convrot_w8a8_gemm_dequant, (q, s, q, s, 32), "x_scale")):
        with pytest.raises(TypeError, match=f"^{name}: need a contiguous torch"):
            f(*args)
        with pytest.raises(TypeError, match="need a torch tensor"):
            f(*[7] * len(args))


_WITHOUT_TORCH = """
import subprocess, sys
sys.path.insert(0, sys.argv[1])
sys.modules["torch"] = None                 # importing it fails
from paper_2512_03673_amd import build
ran = []
def run(cmd, **kw):                         # the compiler's part is left out; what it would write is there
    ran.append(cmd)
    open(cmd[cmd.index("-o") + 1], "w").close()
subprocess.run = run
build.LIB = sys.argv[2]
build.HERE = build.os.path.dirname(build.LIB)
print(build.build(verbose=False, out=build.LIB), len(ran), "torch" in " ".join(map(str, sum(ran, []))))
"""


def test_the_library_builds_without_torch(tmp_path):
    out = tmp_path / "libconvrot.so"
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", _WITHOUT_TORCH, root, str(out)], capture_output=True, text=True, timeout=300)
    from paper_2512_03673_amd import build
    assert r.returncode == 0 and r.stdout.split() == [str(out), str(len(build.SOURCES) + 1), "False"], r.stdout + r.stderr
    assert "_torch_calls.so, which binding.py needs, is not built" in r.stderr and out.exists()


_ANOTHER_LIBRARY = """
import sys
sys.path.insert(0, sys.argv[1])
import torch
from paper_2512_03673_amd import binding as cr
cr.LIB_PATH = sys.argv[2]
try:
    cr.convrot_rotquant_act(torch.zeros(4, 32, dtype=torch.bfloat16), 16)
except TypeError:
    print(sorted({line.split()[-1] for line in open("/proc/self/maps") if "libconvrot" in line}))
"""


def test_the_per_layer_calls_run_in_the_library_that_was_loaded(cr, tmp_path):
    path = shutil.copy(cr.LIB_PATH, tmp_path / "libconvrot_copy.so")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", _ANOTHER_LIBRARY, root, str(path)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == str([str(path)]), r.stdout + r.stderr


class _Refuses(TorchDispatchMode):
    """Every new tensor fails with `error`."""

    def __init__(self, error):
        super().__init__()
        self.error = error

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        if func is torch.ops.aten.empty.memory_format:
            raise self.error
        return func(*args, **(kwargs or {}))


@pytest.mark.parametrize("error", (torch.OutOfMemoryError("no room"), KeyError("who")), ids=lambda e: type(e).__name__)
def test_an_allocation_that_fails_keeps_its_exception(cr, error):
    with FakeTensorMode():      # tensors that say that they are on a GPU
        x = torch.empty(4, 32, dtype=torch.bfloat16, device="cuda")
        q, s = torch.empty(3072, dtype=torch.uint8, device="cuda"), torch.empty(4, device="cuda")
    for f, args in ((cr.convlinear4bit_forward, (x, q, s, 16)), (cr.convlinear8bit_forward, (x, q, s, 16)), (cr.convrot_prepare_weight, (x, 16)),
                    (cr.convrot_rotquant_act8, (x, 16)), (cr.convrot_w4a4_gemm_dequant, (q, s, q, s, 32)),
                    (cr.convrot_w8a8_gemm_dequant, (q, s, q, s, 32))):
        with pytest.raises(type(error)) as caught, _Refuses(error):
            f(*args)
        assert caught.value is error


BAD_OUTPUTS = {"on the host": (TypeError, lambda t: torch.empty(t.shape, dtype=t.dtype)), "transposed": (TypeError, lambda t: t.t()),
               "stretched": (TypeError, lambda t: t[:1, :1].expand(t.shape)), "of another type": (TypeError, lambda t: t.to(torch.float64)),
               "short": (ValueError, lambda t: t[:-1])}


def _calls_with_outputs(cr, m, device):
    """Every call that writes to memory of the caller's: a name, the output as it should be, the call."""
    def new(*shape, dtype=torch.float32):
        return torch.zeros(shape, dtype=dtype, device=device)
    bf16, u8 = torch.bfloat16, torch.uint8
    x, w, xs, ws = new(m, 32, dtype=bf16), new(8, 32, dtype=bf16), new(m), new(8)
    q4, q8 = new(cr.packed_bytes(40, 32), dtype=u8), new(cr.packed_bytes8(40, 32), dtype=u8)
    y, scale = new(m, 8, dtype=bf16), new(m, 1)
    return [
        ("Y", y, lambda o: cr.convlinear4bit_forward(x, q4, ws, 16, Y=o)), ("Y", y, lambda o: cr.convlinear8bit_forward(x, q8, ws, 16, Y=o)),
        ("Y", y, lambda o: cr.convrot_w4a4_gemm_dequant(q4, xs, q4, ws, 32, Y=o)), ("Y", y, lambda o: cr.convrot_w8a8_gemm_dequant(q8, xs, q8, ws, 32, Y=o)),
        ("scale", scale, lambda o: cr.convrot_rotquant_act(x, 16, x_scale=o)), ("scale", scale, lambda o: cr.convrot_rotquant_act8(x, 16, x_scale=o)),
        ("scale", new(8, 1), lambda o: cr.convrot_prepare_weight(w, 16, w_scale=o)), ("scale", new(8, 1), lambda o: cr.convrot_prepare_weight8(w, 16, w_scale=o)),
        ("acc", new(m, 8, dtype=torch.int32), lambda o: cr.convrot_w4a4_gemm_i32(q4, q4, m, 8, 32, acc=o)),
        ("acc", new(m, 8, dtype=torch.int32), lambda o: cr.convrot_w8a8_gemm_i32(q8, q8, m, 8, 32, acc=o)),
        ("codes", new(m, 32, dtype=torch.int8), lambda o: cr.convrot_unpack_codes(q4, m, 32, codes=o)),
        ("out", scale, lambda o: cr.convrot_rotated_absmax(x, 16, 1, out=o)),
    ]


@pytest.mark.parametrize("bad", BAD_OUTPUTS)
def test_rejects_memory_that_it_cannot_write_to(cr, bad):
    error, spoil = BAD_OUTPUTS[bad]
    with FakeTensorMode(allow_non_fake_inputs=True):
        for name, good, call in _calls_with_outputs(cr, 4, "cuda"):
            if good.shape[1] == 1 and bad in ("transposed", "stretched"):       # a vector stays one
                continue
            with pytest.raises(error, match=f"^{name}: need "):
                call(spoil(good))


def test_rejects_a_workspace_and_a_vector_that_are_none(cr):
    with FakeTensorMode(allow_non_fake_inputs=True):
        x, q = torch.empty(4, 32, dtype=torch.bfloat16, device="cuda"), torch.empty(3072, dtype=torch.uint8, device="cuda")
        s, space = torch.empty(4, device="cuda"), torch.empty(64, 256, dtype=torch.uint8, device="cuda")
        for forward in (cr.convlinear4bit_forward, cr.convlinear8bit_forward):
            for bad in ("on the host", "transposed", "stretched"):
                with pytest.raises(TypeError, match="^workspace: need "):
                    forward(x, q, s, 16, workspace=BAD_OUTPUTS[bad][1](space))
            with pytest.raises(ValueError, match="^w_scale: need a vector"):
                forward(x, q, torch.empty(4, 0, device="cuda"), 16)


@pytest.mark.gpu
def test_writes_to_longer_and_raw_memory(cr):
    for name, good, call in _calls_with_outputs(cr, 4, "cuda"):
        size = good.nbytes
        for o in (torch.full((size + 64,), 0x5A, dtype=torch.uint8, device="cuda"), torch.full((size // 4 + 16,), 0x5A5A5A5A, dtype=torch.int32, device="cuda")):
            result = call(o)
            torch.cuda.synchronize()
            assert any(r is o for r in (result if isinstance(result, tuple) else (result,))), name
            assert (o.view(torch.uint8)[:size] != 0x5A).any() and (o.view(torch.uint8)[size:] == 0x5A).all(), name


@pytest.mark.gpu
def test_out_of_device_memory_is_torchs_own_exception(cr):
    n = 1 << 20                 # an output of 2 TB
    x, s = torch.zeros(n, 32, dtype=torch.bfloat16, device="cuda"), torch.ones(n, device="cuda")
    q = torch.zeros(cr.packed_bytes(n, 32), dtype=torch.uint8, device="cuda")
    with pytest.raises(torch.OutOfMemoryError, match="out of memory"):
        cr.convlinear4bit_forward(x, q, s, 16)
    with pytest.raises(torch.OutOfMemoryError, match="out of memory"):
        cr.convrot_w4a4_gemm_dequant(q, s, q, s, 32)


@pytest.mark.gpu
def test_rejects_wrong_shapes_and_statuses(cr):
    dev = dict(device="cuda")
    x, s = torch.zeros(4, 64, dtype=torch.bfloat16, **dev), torch.ones(8, **dev)
    w = torch.zeros(8, 64, dtype=torch.bfloat16, **dev)
    wq, ws = cr.convrot_prepare_weight(w, 16)
    with pytest.raises(ValueError, match="Wq: need 3072 bytes"):
        cr.convlinear4bit_forward(x, wq[:100], ws, 16)
    with pytest.raises(ValueError, match="bias"):
        cr.convlinear4bit_forward(x, wq, ws, 16, bias=torch.zeros(7, dtype=torch.bfloat16, **dev))
    with pytest.raises(TypeError, match="X: need a contiguous"):
        cr.convlinear4bit_forward(x.t(), wq, ws, 16)
    with pytest.raises(ValueError, match="X: need a matrix"):
        cr.convlinear4bit_forward(x[0], wq, ws, 16)
    with pytest.raises(cr.ConvRotError, match="CONVROT_ERR_GROUP"):
        cr.convlinear4bit_forward(x, wq, ws, 17)
    with pytest.raises(cr.ConvRotError, match="CONVROT_ERR_WORKSPACE"):
        cr.convlinear4bit_forward(x, wq, ws, 16, workspace=torch.zeros(256, dtype=torch.uint8, **dev))
    y = torch.empty(4, 8, dtype=torch.bfloat16, **dev)
    assert cr.convlinear4bit_forward(x, wq, ws, 16, Y=y) is y
    q, sc = torch.empty_like(wq), torch.empty_like(s)
    assert cr.convrot_prepare_weight(w, 16, Wq=q, w_scale=sc)[0] is q
    torch.cuda.synchronize()
    assert (y == 0).all() and torch.equal(sc, ws)
