"""What this package is timed on: fused attention forward as a program calls it, `attention(q, k, v, causal)` on
BF16 tensors [B, S, H, 128] that are on the device already, O and LSE coming back.

The sizes are the shapes of `paper_2603_24517_amd/workloads.py` (the paper's prefill grid and the small problem
beside it) and, for what that grid leaves out, generic ones with its head counts: short and ragged prompts, a
chunk of a long prompt against the keys before it, and the few query rows of token-by-token generation.
"""
import math

import torch

import paper_2603_24517_amd as attn

D = 128


def _case(name, B, Hq, Hkv, Sq, Skv, causal, q_mul=1.0, v_uniform=False):
    return {"name": name, "B": B, "Hq": Hq, "Hkv": Hkv, "Sq": Sq, "Skv": Skv, "causal": causal, "q_mul": q_mul,
            "v_uniform": v_uniform}


def listed():
    return [
        # the smallest problem of the workload list: one short sequence, four heads, bidirectional
        _case("mha_full_1x512", 1, 4, 4, 512, 512, False),
        # a batch of short ragged prompts
        _case("mha_causal_24x200", 24, 16, 16, 200, 200, True),
        # one prompt of odd length through a grouped-query layer
        _case("gqa4_causal_1x1111", 1, 32, 8, 1111, 1111, True),
        # two documents through a bidirectional encoder layer
        _case("mha_full_2x1500", 2, 16, 16, 1500, 1500, False),
        # the next 512 tokens of a long prompt against the 16384 keys that end with them
        _case("gqa4_chunk_512_of_16384", 1, 32, 8, 512, 16384, True),
        # generation, one sequence with a long context: one query row against 32768 keys
        _case("gqa4_decode_1x32768", 1, 32, 8, 1, 32768, True),
        # generation, a batch: one query row each against 4000 keys
        _case("gqa4_decode_16x4000", 16, 32, 8, 1, 4000, True),
        # several rows at once per sequence (tokens proposed ahead and checked together)
        _case("gqa8_rows16_2x8192", 2, 64, 8, 16, 8192, True),
        # the headline workload
        _case("mha_full_8x4096", 8, 16, 16, 4096, 4096, False),
        # the same under the causal mask, with peaked softmax rows
        _case("mha_causal_8x4096_q4", 8, 16, 16, 4096, 4096, True, q_mul=4.0),
        # grouped-query prefill of medium length
        _case("gqa4_causal_4x8192", 4, 32, 8, 8192, 8192, True),
        # the longest prefill: 64 query heads on 8 K/V heads
        _case("gqa8_causal_1x32768_vu", 1, 64, 8, 32768, 32768, True, v_uniform=True),
    ]


HEADS = [(16, 16), (32, 8), (32, 4), (64, 8), (4, 4)]     # the head counts of the workload list
MOST_FLOPS = 4.0 * 64 * 32768 * 32768 * D / 2             # the last listed case
MOST_KEYS = 1 << 18                                       # B x Skv of a case of few rows: at most 1 GiB of K and V


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    Hq, Hkv = rng.choice(HEADS)
    kind = rng.choice(["prefill", "prefill", "prefill", "chunk", "few"])
    if kind == "prefill":
        S = _log(rng, 100, 32768)
        B = _log(rng, 1, max(1, 65536 // S)) if S < 65536 else 1
        case = _case("", B, Hq, Hkv, S, S, rng.random() < 0.6, q_mul=rng.choice([1.0, 1.0, 4.0]))
    elif kind == "chunk":
        Sq = _log(rng, 32, 4096)
        Skv = Sq + _log(rng, 64, 32768 - Sq)
        case = _case("", rng.choice([1, 1, 2, 4]), Hq, Hkv, Sq, Skv, True)
    else:
        Sq = rng.choice([1, 1, 1, 2, 4, 7, 16])
        Skv = _log(rng, 256, 32768)
        B = _log(rng, 1, 64)
        case = _case("", max(1, min(B, MOST_KEYS // Skv)), Hq, Hkv, Sq, Skv, True)
    del case["name"]
    while case["B"] > 1 and _flops(case) > MOST_FLOPS:
        case["B"] //= 2
    return case


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, Hq, Hkv, Sq, Skv = (case[k] for k in ("B", "Hq", "Hkv", "Sq", "Skv"))

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)

    q = normal(B, Sq, Hq, D) * case["q_mul"]              # exact: q_mul is a power of two
    k = normal(B, Skv, Hkv, D)
    if case["v_uniform"]:
        v = (torch.rand((B, Skv, Hkv, D), generator=g, device="cuda", dtype=torch.float32) * 2 - 1).to(torch.bfloat16)
    else:
        v = normal(B, Skv, Hkv, D)
    return {"q": q, "k": k, "v": v, "causal": case["causal"]}


def run(state):
    return attn.attention(state["q"], state["k"], state["v"], causal=state["causal"])


def _pairs(case):
    """(query, key) pairs that are not masked, per head."""
    Sq, Skv = case["Sq"], case["Skv"]
    if not case["causal"]:
        return case["B"] * Sq * Skv
    return case["B"] * (Sq * (Skv - Sq) + Sq * (Sq + 1) // 2)


def _flops(case):
    return 4.0 * D * case["Hq"] * _pairs(case)


def work(case):
    B, Hq, Hkv, Sq, Skv = (case[k] for k in ("B", "Hq", "Hkv", "Sq", "Skv"))
    return {"bytes": 2 * D * B * (2 * Hq * Sq + 2 * Hkv * Skv) + 4 * B * Hq * Sq, "flops": _flops(case)}


def tolerance(case):
    # Softmax weights and O are rounded to BF16 once each.  Measured over the listed cases against the same
    # attention in 64 bits, unrounded: O is off by 1.9e-3 .. 2.8e-3 in the 2-norm and by at most 2.6e-2 of the
    # larger of a value and the root mean square (LSE, in FP32 throughout, by 5e-8); four times that.
    return {"rel": 1e-2, "max": 0.1}
