"""The extension module behind the per-layer calls of binding.py: what it rejects before anything is launched."""
import os

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
