"""The kernel with workgroups of four wavefronts, in items of 128 and of 64 rows: edges of its tiles, turns, stages and windows against
the oracle, and the calls that the library itself sends to it."""
import math

import pytest
import torch

import paper_2603_24517_amd as A
from paper_2603_24517_amd import probe as P
import gpu_util as U

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)
ENTRIES = ["always_rows128", "always_rows64"]

# B, Hq, Hkv, Sq, Skv
SHAPES = [
    (1, 1, 1, 1, 1), (1, 1, 1, 128, 32), (1, 1, 1, 129, 33), (1, 1, 1, 65, 64), (1, 2, 1, 63, 65),      # one turn, two
    (1, 1, 1, 128, 96), (1, 1, 1, 128, 128), (2, 1, 1, 100, 160), (1, 1, 1, 64, 192), (1, 1, 1, 64, 224),       # as many turns as stages, one more
    (1, 2, 2, 130, 320), (1, 1, 1, 200, 353), (1, 1, 1, 256, 417), (1, 3, 3, 127, 1025),                # the unrolled loop and what is left over
    (1, 4, 1, 150, 150), (2, 8, 1, 70, 333), (1, 12, 3, 65, 777), (1, 6, 2, 130, 65), (1, 16, 1, 9, 300),       # heads packed 4, 8, 2 to an item
    (1, 2, 2, 300, 200), (1, 1, 1, 700, 130),                                           # causal: rows and whole tiles without keys
    (5, 3, 3, 500, 500), (3, 8, 8, 96, 40), (1, 1, 1, 9000, 40), (13, 40, 40, 33, 35),  # several windows of items, the first one narrower
]


def _entry(name):
    return lambda *a: P.variant_attn_fwd(name, *a)


@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("n", range(len(SHAPES)), ids=lambda n: "x".join(map(str, SHAPES[n])))
def test_parity(n, causal, entry):
    print(f"shape {SHAPES[n]} causal={causal} {entry}", flush=True)
    x = U.rand_qkv(*SHAPES[n], seed=9800 + n, q_mul=4.0 if n % 2 else 1.0)
    U.check_full(*x, causal, SCALE, what=f"{SHAPES[n]}", attn_fwd=_entry(entry))


@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
def test_hard_scores(causal, entry):
    """Scores that outgrow the reference of the first two blocks by far, and both signs of the scale."""
    q, k, v = U.rand_qkv(1, 4, 2, 300, 1500, seed=9900, q_mul=48.0)
    for scale in (SCALE, -SCALE, 0.0):
        U.check_full(q, k, v, causal, scale, what=f"scale={scale}", attn_fwd=_entry(entry))


@pytest.mark.parametrize("entry", ENTRIES)
def test_keys_of_minus_infinite_score(entry):
    """They count for nothing, also where they fill the first blocks of an item or all of a group of wavefronts' blocks."""
    print(entry, flush=True)
    q, k, v = (t.cuda() for t in U.rand_qkv(1, 1, 1, 128, 600, seed=9901))
    q = q.abs()
    live = torch.zeros(600, dtype=torch.bool, device="cuda")
    live[200:230] = live[450:470] = True
    k[:, ~live] = float("-inf")

    def run(k, v):
        o, lse = torch.full_like(q, float("nan")), torch.full((1, 1, 128), float("nan"), device="cuda")
        assert _entry(entry)(q, k, v, o, lse, 1, 1, 1, 128, k.shape[1], 128, False, SCALE, torch.cuda.current_stream().cuda_stream) == 0
        return o.float(), lse

    o, lse = run(k, v)
    U.check_full(q.cpu(), k[:, live].contiguous().cpu(), v[:, live].contiguous().cpu(), False, SCALE, what="the others alone",
                 attn_fwd=_entry(entry))
    ref, ref_lse = run(k[:, live].contiguous(), v[:, live].contiguous())
    # both are within two roundings to BF16 of the exact result
    assert (o - ref).abs().max() <= 2.0 ** -7 * ref.abs().max()
    assert torch.allclose(lse, ref_lse, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("shape,causal", [((1, 32, 8, 1111, 1111), True), ((24, 16, 16, 200, 200), True), ((44, 4, 4, 300, 300), False),
                                          ((2, 16, 16, 1201, 1300), True)])
def test_as_shipped(shape, causal):
    """Calls that the library sends there itself are no further from the exact result than in items of 256 rows, and the same from one launch
    to the next."""
    print(f"shape {shape} causal={causal}", flush=True)
    q, k, v = U.rand_qkv(*shape, seed=9950 + shape[0])
    dev = [t.cuda() for t in (q, k, v)]

    def run(entry):
        (B, Sq, Hq, D), (_, Skv, Hkv, _) = q.shape, k.shape
        o, lse = torch.full_like(dev[0], float("nan")), torch.full((B, Hq, Sq), float("nan"), device="cuda")
        fwd = A.attn_fwd if entry is None else _entry(entry)
        assert fwd(*dev, o, lse, B, Hq, Hkv, Sq, Skv, D, causal, SCALE, torch.cuda.current_stream().cuda_stream) == 0
        return o, lse

    o, lse = run(None)
    assert any(torch.equal(o, run(e)[0]) for e in ENTRIES)
    for _ in range(3):
        again = run(None)
        assert torch.equal(o, again[0]) and torch.equal(lse, again[1])
    (B, Sq, Hq, D), (_, Skv, Hkv, _) = q.shape, k.shape
    exact = torch.empty(o.shape, dtype=torch.float64, device="cuda")
    for b in range(B):
        for h in range(Hq):
            s = SCALE * (dev[0][b, :, h].double() @ dev[1][b, :, h // (Hq // Hkv)].double().T)
            if causal:
                s = s.masked_fill(torch.ones(Sq, Skv, dtype=torch.bool, device="cuda").triu(Skv - Sq + 1), float("-inf"))
            exact[b, :, h] = torch.softmax(s, -1) @ dev[2][b, :, h // (Hq // Hkv)].double()
    err, err256 = ((x.double() - exact).norm().item() for x in (o, run("whole_items")[0]))
    print(f"error {err / exact.norm().item():.3e}, in items of 256 rows {err256 / exact.norm().item():.3e}", flush=True)
    assert err <= 1.01 * err256         # (more than 10^6 roundings each: their sums differ by far less than 1 % between two draws)
