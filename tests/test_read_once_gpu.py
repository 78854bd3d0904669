"""Few rows against keys and values that are read once, past the caches, in rounds of parts where whole items would leave a round partly empty:
the oracle's rows, and the bits of the path without device memory, on the null stream, on another one and from a graph."""
import math

import numpy as np
import pytest
import torch

import paper_2603_24517_amd as A
import gpu_util as U
import test_shared_bits_gpu as T

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)


# B, Hq, Hkv, Sq, Skv: rounds of parts (272, 264, 144 and 560 items), and shared items that go past the caches on the null stream alone
ROUNDS = [(17, 16, 16, 1, 2711), (33, 32, 8, 2, 2711), (9, 16, 16, 7, 8200), (280, 16, 2, 1, 2811)]
REGION = [(1, 32, 8, 1, 32768), (16, 32, 8, 2, 1811)]


@pytest.mark.parametrize("shape", ROUNDS + REGION, ids=lambda s: "x".join(map(str, s)))
def test_rounds_of_parts(shape):
    print(f"shape {shape}", flush=True)
    B, Hq, Hkv, Sq, Skv = shape
    x = U.rand_qkv(*shape, seed=9970 + B)
    rng = np.random.default_rng(B)
    rows = np.stack([rng.integers(0, n, 64) for n in (B, Hq, Sq)], axis=1)
    rows[0], rows[1] = (0, 0, 0), (B - 1, Hq - 1, Sq - 1)
    for causal in (False, True):
        U.check_rows(*x, rows, causal, SCALE, what=f"{shape} causal={causal}")
    dev = tuple(t.cuda() for t in x)
    ref = T._run(dev, True, "no_pool")
    for rep in range(3):
        assert T._same(T._run(dev, True), ref), rep
    out = torch.empty_like(ref[0]), torch.empty_like(ref[1])
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()

    def launch():
        rc = A.attn_fwd(*dev, *out, B, Hq, Hkv, Sq, Skv, 128, True, SCALE, side.cuda_stream)
        assert rc == 0, A.attn_strerror(rc)

    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        launch()
    for rep in range(6):
        for t in out:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay() if rep % 2 else launch()
        torch.cuda.synchronize()
        assert T._same(out, ref), rep
