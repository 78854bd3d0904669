"""Items of the 256-row kernel that several workgroups share: where an item is cut, the merge of the parts, and the path
for a launch that finds no device memory for them."""
import math

import pytest
import torch

import paper_2603_24517_amd as A
from paper_2603_24517_amd import probe as P
import gpu_util as U

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)

# B, Hq, Hkv, Sq, Skv
SHAPES = [
    (1, 1, 1, 1, 1), (1, 1, 1, 256, 64), (1, 2, 1, 257, 129),      # items of 1 .. 3 blocks: never cut
    (1, 1, 1, 256, 256), (1, 1, 1, 300, 1025),                     # the shortest that is, one item in all; a partial last block
    (2, 8, 2, 130, 777), (1, 6, 2, 520, 1999), (1, 8, 1, 65, 4097),
    (3, 2, 2, 1111, 1111), (1, 2, 1, 2600, 900),                   # causal: rows and whole items without keys
    (1, 1, 1, 17000, 320),                                         # 67 tiles in a group: more than a wavefront has lanes
    (5, 16, 4, 500, 500), (24, 16, 16, 65, 200),                   # 160 and 384 items
]


def _inputs(n, q_mul=1.0):
    return U.rand_qkv(*SHAPES[n], seed=9300 + n, q_mul=q_mul)


def _entry(name):
    return None if name is None else (lambda *a: P.variant_attn_fwd(name, *a))


@pytest.mark.parametrize("entry", ["always_share", "always_share_no_pool"])
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("n", range(len(SHAPES)), ids=lambda n: "x".join(map(str, SHAPES[n])))
def test_parity(n, causal, entry):
    print(f"shape {SHAPES[n]} causal={causal} {entry}", flush=True)
    U.check_full(*_inputs(n, q_mul=4.0 if n % 2 else 1.0), causal, SCALE, what=f"{SHAPES[n]}", attn_fwd=_entry(entry))


@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
def test_hard_scores(causal):
    q, k, v = U.rand_qkv(1, 4, 2, 300, 1500, seed=9400, q_mul=48.0)
    for scale in (SCALE, -SCALE, 0.0):
        U.check_full(q, k, v, causal, scale, what=f"scale={scale}", attn_fwd=_entry("always_share"))


def test_keys_of_minus_infinite_score():
    """Keys whose score is minus infinity count for nothing, also where they fill whole parts of an item."""
    q, k, v = U.rand_qkv(1, 1, 1, 256, 2048, seed=9401)
    q = q.abs()
    k[:, 200:] = float("-inf")
    o, lse = torch.empty_like(q.cuda()), torch.empty((1, 1, 256), device="cuda")
    rc = P.variant_attn_fwd("always_share", q.cuda(), k.cuda(), v.cuda(), o, lse, 1, 1, 1, 256, 2048, 128, False, SCALE,
                            torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    U.check_full(q, k[:, :200].contiguous(), v[:, :200].contiguous(), False, SCALE, what="the finite keys alone")
    ref, ref_lse = A.attention(q.cuda(), k[:, :200].contiguous().cuda(), v[:, :200].contiguous().cuda(), causal=False)
    # both are within two roundings to BF16 of the exact result
    assert (o.float() - ref.float()).abs().max() <= 2.0 ** -7 * ref.float().abs().max()
    assert torch.allclose(lse, ref_lse, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("entry", ["always_share", "always_share_no_pool"])
def test_many_streams_at_once_and_graph_replay(entry):
    """Launches in flight together, items in two parts and in four, do not touch each other's parts: each gives the bits of
    a launch alone on the device.  Nine launches of 10, 14 and 11 units are more than the 64 serve at a time."""
    shapes = [(1, 16, 4, 600, 6000), (2, 16, 16, 1025, 5000), (1, 32, 8, 512, 8192)] * 3
    xs = [tuple(t.cuda() for t in U.rand_qkv(*s, seed=9500 + i)) for i, s in enumerate(shapes)]
    outs = [(torch.empty_like(x[0]), torch.empty((x[0].shape[0], x[0].shape[2], x[0].shape[1]), device="cuda")) for x in xs]

    def launch(x, o, stream, entry):
        (B, Sq, Hq, D), (_, Skv, Hkv, _) = x[0].shape, x[1].shape
        rc = _entry(entry)(*x, *o, B, Hq, Hkv, Sq, Skv, D, True, SCALE, stream.cuda_stream)
        assert rc == 0, A.attn_strerror(rc)

    ref = []
    for n, (x, o) in enumerate(zip(xs, outs)):
        launch(x, o, torch.cuda.current_stream(), "always_share")
        torch.cuda.synchronize()
        ref.append([t.clone() for t in o])
        launch(x, o, torch.cuda.current_stream(), "whole_items")
        torch.cuda.synchronize()
        whole = o[0].float()
        launch((x[0], x[1], x[2].abs()), o, torch.cuda.current_stream(), "whole_items")
        torch.cuda.synchronize()
        # On either side a weight is rounded to BF16 (2^-9 of it), and with it the sum that O is divided by, then O (2^-9)
        assert ((ref[n][0].float() - whole).abs() <= 2.0 ** -7 * o[0].float() + 2.0 ** -8 * whole.abs() + 1e-6).all(), n
        assert torch.allclose(ref[n][1], o[1], rtol=1e-5, atol=1e-5), n
    streams = [torch.cuda.Stream() for _ in xs]
    graphs = []
    for x, o, s in zip(xs, outs, streams):
        launch(x, o, s, entry)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            launch(x, o, s, entry)
        graphs.append(g)
    for rep in range(20):
        for o in outs:
            o[0].fill_(float("nan"))
            o[1].fill_(float("nan"))
        torch.cuda.synchronize()
        for x, o, s, g in zip(xs, outs, streams, graphs):
            with torch.cuda.stream(s):
                g.replay() if rep % 2 else launch(x, o, s, entry)
        torch.cuda.synchronize()
        for n, (o, r) in enumerate(zip(outs, ref)):
            assert torch.equal(o[0], r[0]) and torch.equal(o[1], r[1]), (rep, n)
