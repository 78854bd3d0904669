"""attention(): its native call and its general form give what the C entry gives, on the stream that is current, and refuse the same."""
import math

import pytest
import torch

import paper_2603_24517_amd as A
import gpu_util as U

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)
SHAPE = (2, 8, 2, 100, 333)


class Sub(torch.Tensor):
    pass


def _same(a, b):
    return torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("causal", [False, True])
def test_forms_agree(causal):
    q, k, v = (t.cuda() for t in U.rand_qkv(*SHAPE, seed=9960))
    B, Hq, Hkv, Sq, Skv = SHAPE
    ref = torch.empty_like(q), torch.empty((B, Hq, Sq), device="cuda")
    assert A.attn_fwd(q, k, v, *ref, B, Hq, Hkv, Sq, Skv, 128, causal, SCALE, torch.cuda.current_stream().cuda_stream) == 0
    out = A.attention(q, k, v, causal=causal)
    assert type(out) is tuple and out[0].dtype == torch.bfloat16 and out[1].dtype == torch.float32 and _same(out, ref)
    for scale in (SCALE, torch.tensor(SCALE, dtype=torch.float64), str(SCALE)):
        assert _same(A.attention(q, k, v, int(causal), scale), ref)
    assert _same(A._attention(q, k, v, causal, None), ref)
    assert _same(A.attention(q.as_subclass(Sub), k, v, causal), ref)
    assert _same(A.attention(torch.nn.Parameter(q), k, v, causal), ref)
    with torch.device("cpu"):                   # a torch function mode
        assert _same(A.attention(q, k, v, causal), ref)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        out = A.attention(q, k, v, causal)
    torch.cuda.current_stream().wait_stream(side)
    assert _same(out, ref)


def test_calls_that_are_refused():
    q, k, v = (t.cuda() for t in U.rand_qkv(*SHAPE, seed=9961))
    for bad in ((q.cpu(), k, v), (q.float(), k, v), (q, k.transpose(1, 2), v), (q[0], k, v), (q, k, v[:, 1:].contiguous()), (q, k[:1], v[:1])):
        for f in (A.attention, lambda *a: A._attention(*a, False, None)):
            with pytest.raises(ValueError):
                f(*bad)
    with pytest.raises(A.AttnError) as e:
        A.attention(q[..., :64].contiguous(), k[..., :64].contiguous(), v[..., :64].contiguous())
    assert e.value.code == A.ATTN_E_UNSUPPORTED
    with pytest.raises(A.AttnError) as e:
        A.attention(q, k, v, scale=float("nan"))
    assert e.value.code == A.ATTN_E_SCALE
    with pytest.raises(AttributeError):
        A.attention(None, k, v)
    with pytest.raises(RuntimeError):           # no storage behind a batched tensor
        torch.vmap(lambda x: A.attention(x, k, v)[0])(q[None])
