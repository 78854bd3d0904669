"""attention()'s native call and exceptions that torch raises inside it, on tensors without storage."""
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from torch.utils._python_dispatch import TorchDispatchMode

import paper_2603_24517_amd as A


class Refuse(TorchDispatchMode):
    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        if func is torch.ops.aten.empty_like.default:
            raise KeyError("no")
        return func(*args, **(kwargs or {}))


@pytest.mark.parametrize("mode,error", [(Refuse, KeyError), (FakeTensorMode, AssertionError)])
def test_exception_of_a_dispatch_mode_reaches_the_caller(mode, error):
    with FakeTensorMode():
        fake = [torch.empty(1, 4, 2, 128, device="cuda", dtype=torch.bfloat16) for _ in range(3)]
    q, k, v = (torch._to_functional_tensor(t) for t in fake)       # (torch.Tensor itself, on a device, as the native call wants them)
    A._load_call()
    with mode(), pytest.raises(error):
        A.attention(q, k, v)


class OnDevice:
    """What the general form asks of a tensor."""
    is_cuda, dtype, device = True, torch.bfloat16, "cuda:0"

    def __init__(self, *shape):
        self.shape = shape

    is_contiguous, dim, get_device, data_ptr = (lambda self: True), (lambda self: 4), (lambda self: 0), (lambda self: 64)


@pytest.mark.parametrize("current", [0, 1])
def test_general_form_on_the_current_device_needs_neither_stream_object_nor_device_context(monkeypatch, current):
    """It serves every call under torch.set_default_device(), a function mode: where q's device is the current one, the two took longer than the rest of it."""
    log = []

    class Context:
        def __init__(self, index):
            log.append(index)

        __enter__ = __exit__ = lambda self, *a: None

    class Lib:
        attn_fwd = staticmethod(lambda *a: log.append(a[-1]) or A.ATTN_OK)

    monkeypatch.setattr(A, "load", lambda: Lib)
    monkeypatch.setattr(torch, "empty_like", lambda t: t)
    monkeypatch.setattr(torch, "empty", lambda *a, **k: OnDevice(1, 2, 4))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: current)
    monkeypatch.setattr(torch.cuda, "device", Context)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: pytest.fail("a Stream object"))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 7 + index)
    x = OnDevice(1, 4, 2, 128)
    A._attention(x, x, x, False, None)
    assert log == ([7] if current == 0 else [0, 7])
