"""Calls of few query rows and many work items, on both sides of the rules that choose their kernel."""
import math

import pytest
import torch

import paper_2603_24517_amd as A

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)


@pytest.mark.parametrize("B", [65535, 65536])
def test_one_key_and_the_most_workgroups_of_a_launch(B):
    """One row and one key per head: O is V bit for bit and LSE the one score.  65535 x 128 items are the most that a
    launch of one workgroup per item can have."""
    print(f"B={B}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(B)
    q, k, v = (torch.empty((B, 1, 128, 128), dtype=torch.bfloat16, device="cuda").normal_(generator=g) for _ in range(3))
    o, lse = A.attention(q, k, v, causal=True)
    assert torch.equal(o, v)
    for b in range(0, B, 8192):
        s = SCALE * (q[b:b + 8192, 0].float() * k[b:b + 8192, 0].float()).sum(-1)
        # 128 products, exact in FP32, added up in another order: at most 128 roundings of a sum below 128 x |q||k|
        assert torch.allclose(lse[b:b + 8192, :, 0], s, rtol=1e-5, atol=1e-4), b
