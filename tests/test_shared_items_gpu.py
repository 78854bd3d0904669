"""Items of the split-key kernel that several workgroups share: partial results through device memory, the pool
that memory comes from, and the path without it."""
import math

import numpy as np
import pytest
import torch

import paper_2603_24517_amd as A
from paper_2603_24517_amd import probe as P
import gpu_util as U

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)

# B, Hq, Hkv, Sq, Skv: items x parts <= 256, from 40 blocks of 32 keys on (54 with more than 85 items, 66 with more than 2 tiles)
SHAPES = [
    (1, 1, 1, 1, 1248), (1, 1, 1, 1, 1249), (1, 8, 1, 4, 1280), (1, 8, 1, 5, 1281),   # 39 and 40 blocks, full and ragged; 32 and 40 rows
    (1, 32, 8, 1, 3001), (2, 6, 2, 7, 5000), (1, 4, 4, 33, 2049), (3, 16, 2, 16, 2199),
    (1, 1, 1, 1, 65537), (16, 32, 8, 1, 1800), (17, 32, 8, 1, 1800),                  # most parts; 128 items in two parts, 136 in one
    (40, 32, 8, 2, 700),                                                              # few rows, more items than compute units
]


def _inputs(n, q_mul=1.0):
    return U.rand_qkv(*SHAPES[n], seed=9100 + n, q_mul=q_mul)


@pytest.mark.parametrize("entry", [None, "no_pool"])
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("n", range(len(SHAPES)), ids=lambda n: "x".join(map(str, SHAPES[n])))
def test_parity(n, causal, entry):
    print(f"shape {SHAPES[n]} causal={causal} {entry}", flush=True)
    fwd = None if entry is None else (lambda *a: P.variant_attn_fwd(entry, *a))
    U.check_full(*_inputs(n, q_mul=4.0 if n % 2 else 1.0), causal, SCALE, what=f"{SHAPES[n]}", attn_fwd=fwd)


def test_hard_scores():
    q, k, v = U.rand_qkv(1, 4, 2, 3, 4000, seed=9200, q_mul=48.0)
    for scale in (SCALE, -SCALE, 0.0):
        U.check_full(q, k, v, True, scale, what=f"scale={scale}")
    q, k, v = U.rand_qkv(1, 2, 2, 2300, 2000, seed=9201)          # rows without keys, tiles without keys among them
    U.check_full(q, k, v, True, SCALE, what="empty rows")


def _launch(x, out, stream, entry=None):
    q, k, v = x
    (B, Sq, Hq, D), (_, Skv, Hkv, _) = q.shape, k.shape
    rc = (A.attn_fwd if entry is None else lambda *a: P.variant_attn_fwd(entry, *a))(q, k, v, out[0], out[1], B, Hq, Hkv, Sq, Skv, D, True, SCALE, stream.cuda_stream)
    assert rc == 0, A.attn_strerror(rc)


@pytest.mark.parametrize("entry", [None, "no_pool"])
def test_many_streams_at_once_and_graph_replay(entry):
    """Launches in flight together do not touch each other's partial results, and give their units back.  Without units
    (no_pool) a workgroup that starts after its item's result is stored finds that result, and nothing to do."""
    xs = [tuple(t.cuda() for t in _inputs(n)) for n in (4, 5, 7, 9)] * 2
    outs = [(torch.empty_like(x[0]), torch.empty((x[0].shape[0], x[0].shape[2], x[0].shape[1]), device="cuda")) for x in xs]
    ref = []
    for x, o in zip(xs, outs):
        _launch(x, o, torch.cuda.current_stream(), entry)
        torch.cuda.synchronize()
        ref.append([t.clone() for t in o])
    streams = [torch.cuda.Stream() for _ in xs]
    graphs = []
    for x, o, s in zip(xs, outs, streams):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            _launch(x, o, s, entry)
        graphs.append(g)
    for rep in range(40):           # (a run of units that stayed taken would use the pool up)
        for o in outs:
            o[0].fill_(float("nan"))
            o[1].fill_(float("nan"))
        torch.cuda.synchronize()
        for x, o, s, g in zip(xs, outs, streams, graphs):
            with torch.cuda.stream(s):
                g.replay() if rep % 2 else _launch(x, o, s, entry)
        torch.cuda.synchronize()
        for n, (o, r) in enumerate(zip(outs, ref)):
            assert torch.equal(o[0], r[0]) and torch.equal(o[1], r[1]), (rep, n)
