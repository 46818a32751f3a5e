"""The native half of the binding without a GPU: tensors that have no memory to point at, and arguments that are refused,
end in the Python exception they ended in when the marshalling was Python."""
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

import paper_2506_05413_amd as sr
from paper_2506_05413_amd import binding


def device_tensors(M=4, K=128, N=32):
    """Shapes and types of device tensors; no memory behind them."""
    with FakeTensorMode():
        e = lambda shape, dtype: torch.empty(shape, dtype=dtype, device="cuda")
        return dict(X=e((M, K), torch.float16), q=e((M, K // 2), torch.uint8), s=e((M,), torch.float32),
                    W=e((N, K // 2), torch.uint8), ws=e((N,), torch.float32), Y=e((M, N), torch.float16),
                    X6=e((768 * K // 128,), torch.uint8), W6=e((768 * N // 8 * K // 128,), torch.uint8),
                    work=e((1 << 20,), torch.uint8), kq=e((M, K // 2), torch.uint8), ks=e((M, 1), torch.float32))


CALLS = {
    "act": lambda t, x: sr.sr_fwht_quant_act(x, None, 0.9, t["q"], t["s"]),
    "heads": lambda t, x: sr.sr_fwht_quant_act_heads(x, 4, True, None, 0.9, t["q"], t["s"]),
    "act_f6": lambda t, x: sr.sr_fwht_quant_act_f6(x, None, 0.9, t["X6"], t["s"]),
    "gate": lambda t, x: sr.sr_swiglu_fwht_quant_act(x, t["X"], None, 0.9, t["q"], t["s"]),
    "decode": lambda t, x: sr.sr_w4a4_linear_decode(x, None, t["W"], t["ws"], 0.9, t["Y"], workspace=t["work"]),
    "kv": lambda t, x: sr.sr_kv_quant_asym(x, 128, 0.95, t["kq"], t["ks"], t["ks"]),
}


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
@pytest.mark.parametrize("name", CALLS)
def test_tensor_without_memory_inside_vmap(name):
    """The address is asked for before the interpreter's lock is given up: asked for behind it, the C++ exception left with
    the lock not held, which ends the process."""
    t = device_tensors()

    def call(x):
        CALLS[name](t, x)
        return x

    with FakeTensorMode():
        batch = torch.empty((3, 4, 128), dtype=torch.float16, device="cuda")
    with pytest.raises(RuntimeError, match="(?i)storage|data pointer"):
        torch.func.vmap(call)(batch)


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
def test_torch_exceptions_keep_their_type():
    t = device_tensors()
    with FakeTensorMode():
        scalar = torch.empty((), dtype=torch.float16, device="cuda")
    with pytest.raises(IndexError):
        sr.sr_w4a4_gemm(t["q"], t["s"], t["W"], t["ws"], Y=scalar)


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
def test_offline_calls_do_without_the_native_half(monkeypatch):
    """Calibration, fold and repacking marshal through ctypes and need no module that is tied to one torch."""
    class Stream:
        cuda_stream = 0

    def unavailable():
        raise ImportError("not built for this torch")

    monkeypatch.setattr(binding, "_native", None)
    monkeypatch.setattr(binding, "_marshal", unavailable)
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    t = device_tensors()
    with FakeTensorMode():
        W, f = torch.empty((128, 32), dtype=torch.float16, device="cuda"), torch.empty(128, device="cuda")
        for call in (lambda: sr.sr_calib_absmax(t["X"], f), lambda: sr.sr_pack_f6_tiles(t["W"], t["W6"]),
                     lambda: sr.sr_fold_smooth_rotate_quant(W, f, 0.5)):
            with pytest.raises(sr.SmoothRotError):       # the library is reached and refuses the missing memory
                call()


def test_native_half_of_another_torch_is_refused(monkeypatch):
    monkeypatch.setattr(binding, "_native", None)
    monkeypatch.setattr(torch, "__version__", "0.0.1")
    with pytest.raises(ImportError, match="0.0.1"):
        sr.sr_fwht_quant_act(None, None)


@pytest.mark.gpu
@pytest.mark.parametrize("call", [lambda x: sr.sr_fwht_quant_act(x, None), lambda x: sr.sr_kv_quant_asym(x, 64)])
def test_out_of_memory_is_torchs(gpu, call):
    """The outputs of 2^37 rows of 64 values do not fit: torch.OutOfMemoryError, which a server catches to shed load."""
    x = torch.zeros((1, 64), dtype=torch.float16, device="cuda").expand(1 << 37, 64)
    with pytest.raises(torch.OutOfMemoryError):
        call(x)
    q, s = gpu.sr_fwht_quant_act(x[:2].contiguous(), None)
    assert bool((s == 1).all()) and not bool(q.any())
