"""Launches with shared items on the null stream, which have memory of their own, give the bits of those on other streams, which take
theirs from the pool, however calls of both kernels and of several sizes follow one another."""
import math
import random

import pytest
import torch

import paper_2603_24517_amd as A
import gpu_util as U

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)

# B, Hq, Hkv, Sq, Skv: split-key kernel (20 parts, 2, 4 of 256 workgroups), 256-row kernel (4 parts, 2, 22)
CALLS = [(1, 32, 8, 1, 32768), (16, 32, 8, 1, 4000), (2, 64, 8, 16, 8192), (1, 32, 8, 512, 8192), (5, 12, 3, 2326, 2326), (1, 4, 4, 700, 40001)]


def test_both_kernels_in_turn():
    assert torch.cuda.current_stream().cuda_stream == 0
    xs = [tuple(t.cuda() for t in U.rand_qkv(*s, seed=9990 + i)) for i, s in enumerate(CALLS)]
    outs = [(torch.empty_like(x[0]), torch.empty((x[0].shape[0], x[0].shape[2], x[0].shape[1]), device="cuda")) for x in xs]
    side = torch.cuda.Stream()

    def run(i, stream):
        B, Hq, Hkv, Sq, Skv = CALLS[i]
        assert A.attn_fwd(*xs[i], *outs[i], B, Hq, Hkv, Sq, Skv, 128, True, SCALE, stream) == 0
        return outs[i]

    torch.cuda.synchronize()
    ref = []
    for i in range(len(CALLS)):
        run(i, side.cuda_stream)
        torch.cuda.synchronize()
        ref.append([t.clone() for t in outs[i]])
    rng = random.Random(5)
    order = [rng.randrange(len(CALLS)) for _ in range(120)]
    for lo in range(0, len(order), 6):
        for o in outs:
            for t in o:
                t.fill_(float("nan"))
        for i in order[lo:lo + 6]:
            run(i, 0)
        torch.cuda.synchronize()
        for i in set(order[lo:lo + 6]):
            assert torch.equal(outs[i][0], ref[i][0]) and torch.equal(outs[i][1], ref[i][1]), (lo, CALLS[i])
