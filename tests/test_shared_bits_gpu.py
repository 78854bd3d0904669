"""Items shared among workgroups give the same bits whatever the order in which the workgroups arrive, and whether or not
the launch finds device memory for their partial results."""
import math

import pytest
import torch

import paper_2603_24517_amd as A
from paper_2603_24517_amd import probe as P
import gpu_util as U
import test_shared_items_gpu as I
import test_shared_rows_gpu as R

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)


@pytest.fixture(params=["null_stream", "other_stream"], autouse=True)
def stream(request):
    """The null stream's launches have memory of their own for the parts, others take units of the pool."""
    if request.param == "null_stream":
        assert torch.cuda.current_stream().cuda_stream == 0
        yield
    else:
        with torch.cuda.stream(torch.cuda.Stream()):
            assert torch.cuda.current_stream().cuda_stream != 0
            yield
    torch.cuda.synchronize()


def _run(x, causal, entry=None, scale=SCALE):
    q, k, v = x
    (B, Sq, Hq, D), (_, Skv, Hkv, _) = q.shape, k.shape
    o, lse = torch.full_like(q, float("nan")), torch.full((B, Hq, Sq), float("nan"), device="cuda")
    fwd = A.attn_fwd if entry is None else (lambda *a: P.variant_attn_fwd(entry, *a))
    rc = fwd(q, k, v, o, lse, B, Hq, Hkv, Sq, Skv, D, causal, scale, torch.cuda.current_stream().cuda_stream)
    assert rc == 0, A.attn_strerror(rc)
    return o, lse


def _same(a, b):
    return torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])


@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("n", range(len(I.SHAPES)), ids=lambda n: "x".join(map(str, I.SHAPES[n])))
def test_split_key_kernel(n, causal):
    print(f"shape {I.SHAPES[n]} causal={causal}", flush=True)
    x = tuple(t.cuda() for t in I._inputs(n, q_mul=4.0 if n % 2 else 1.0))
    ref = _run(x, causal, "no_pool")
    assert torch.isfinite(ref[0]).all()
    for rep in range(5):
        assert _same(_run(x, causal), ref), rep


def test_split_key_kernel_hard_scores():
    x = tuple(t.cuda() for t in U.rand_qkv(1, 4, 2, 3, 4000, seed=9200, q_mul=48.0))
    for scale in (SCALE, -SCALE, 0.0):
        assert _same(_run(x, True, None, scale), _run(x, True, "no_pool", scale)), scale


@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("n", range(len(R.SHAPES)), ids=lambda n: "x".join(map(str, R.SHAPES[n])))
def test_256_row_kernel(n, causal):
    print(f"shape {R.SHAPES[n]} causal={causal}", flush=True)
    x = tuple(t.cuda() for t in R._inputs(n, q_mul=4.0 if n % 2 else 1.0))
    ref = _run(x, causal, "always_share_no_pool")
    assert torch.isfinite(ref[0]).all()
    for rep in range(5):
        assert _same(_run(x, causal, "always_share"), ref), rep


# B, Hq, Hkv, Sq, Skv: what the library itself shares, 555 items to 12 on 256 workgroups: two parts at most, three, four, six, 22; tiles
# of one row, heads packed eight to an item
SHARED_CALLS = [(5, 12, 3, 2326, 2326), (2, 16, 16, 1025, 5000), (1, 32, 8, 512, 8192), (1, 16, 2, 700, 20001), (1, 4, 4, 700, 40001)]


@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("shape", SHARED_CALLS, ids=lambda s: "x".join(map(str, s)))
def test_256_row_kernel_as_shipped(shape, causal):
    print(f"shape {shape} causal={causal}", flush=True)
    x = tuple(t.cuda() for t in U.rand_qkv(*shape, seed=9600 + shape[0], q_mul=2.0))
    ref = _run(x, causal, "no_pool")
    whole = _run(x, causal, "whole_items")
    assert not torch.equal(ref[0], whole[0])        # (it is shared: parts round their weights against references of their own)
    for rep in range(20):
        assert _same(_run(x, causal), ref), rep


@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
def test_256_row_kernel_hard_scores(causal):
    x = tuple(t.cuda() for t in U.rand_qkv(1, 4, 2, 300, 1500, seed=9400, q_mul=48.0))
    for scale in (SCALE, -SCALE, 0.0):
        assert _same(_run(x, causal, "always_share", scale), _run(x, causal, "always_share_no_pool", scale)), scale
