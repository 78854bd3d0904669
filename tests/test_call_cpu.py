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
