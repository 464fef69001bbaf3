"""Performance cases of the attention library, through its public Python entry points.

`listed()` holds the fixed cases, `draw(rng)` gives further ones of the same ranges.  A case is a plain dict;
its "kind" names the entry point:

    fwd    sdpa            square attention: prefill or training forward, optionally causal, optionally with the
                           log-sum-exp that the backward pass needs
    kv     sdpa_kv         a block of queries against a dense KV cache (decoding step, prefill chunk), grouped heads,
                           optionally a length per batch entry
    paged  sdpa_paged      the same against a paged cache
    bwd    sdpa_backward   gradients of q, k, v, grouped heads included

Values are standard normals in the 16-bit input type, as in the library's benchmark; "qk_std" widens Q and K where
the benchmark's own long-context FP16 configuration does.
"""
import math

import torch

from paper_2603_01960_amd import binding as lib

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


def listed():
    return [
        # the benchmark's smallest configuration: one short prompt, two heads; host time and one launch
        dict(name="fwd_smallest", kind="fwd", B=1, H=2, S=128, D=64, dtype="f16", causal=False, lse=False),
        # the benchmark's text regime
        dict(name="fwd_text", kind="fwd", B=4, H=16, S=1024, D=64, dtype="f16", causal=False, lse=False),
        # the benchmark's vision regime: 196 patches and a class token, a length that no tile divides
        dict(name="fwd_vision", kind="fwd", B=64, H=12, S=197, D=64, dtype="bf16", causal=False, lse=False),
        # the benchmark's long-context regime (its default workload)
        dict(name="fwd_long", kind="fwd", B=2, H=32, S=8192, D=128, dtype="bf16", causal=False, lse=False),
        # a point of the benchmark's S x D grid: training forward under the causal mask, log-sum-exp kept
        dict(name="fwd_grid_causal", kind="fwd", B=4, H=16, S=2048, D=96, dtype="f16", causal=True, lse=True),
        # one sequence being decoded: 32 query heads over 8 key/value heads, 8192 cached keys
        dict(name="decode_single", kind="kv", B=1, H=32, Hkv=8, Sq=1, Skv=8192, D=128, dtype="bf16", causal=False, fill=1.0),
        # a batch being decoded from a paged cache, every sequence at a length of its own
        dict(name="decode_batch_paged", kind="paged", B=32, H=32, Hkv=8, Sq=1, Skv=8192, D=128, dtype="bf16", causal=False,
             fill=0.25, block_rows=128),
        # a chunk of 512 new tokens per sequence against what is cached so far
        dict(name="prefill_chunk", kind="kv", B=4, H=32, Hkv=8, Sq=512, Skv=8192, D=128, dtype="bf16", causal=True, fill=0.5),
        # the vision, text and long-context regimes trained: their backward passes
        dict(name="bwd_vision", kind="bwd", B=64, H=12, Hkv=12, S=197, D=64, dtype="bf16", causal=False),
        dict(name="bwd_text_causal", kind="bwd", B=4, H=16, Hkv=16, S=1024, D=64, dtype="f16", causal=True),
        dict(name="bwd_long", kind="bwd", B=2, H=32, Hkv=32, S=8192, D=128, dtype="bf16", causal=False),
        # a grid point trained with grouped heads at the widest head dimension
        dict(name="bwd_grouped_wide", kind="bwd", B=4, H=16, Hkv=4, S=2048, D=160, dtype="bf16", causal=True),
    ]


# what one drawn case may cost at most: the work of the long-context forward pass
MOST_FLOPS = 2.2e12
MOST_BYTES = 8e8


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _length(rng, lo, hi):
    """A length spread over the logarithm of its range; a third of them round numbers, the rest as they fall."""
    n = _log_int(rng, lo, hi)
    if rng.random() < 0.34 and n >= 64:
        n = 1 << (n.bit_length() - 1)
    return n


def draw(rng):
    while True:
        kind = rng.choice(["fwd", "fwd", "fwd", "kv", "kv", "paged", "bwd", "bwd"])
        case = dict(kind=kind, dtype=rng.choice(["f16", "bf16"]), D=rng.choice([64, 96, 128, 160]))
        if kind in ("fwd", "bwd"):
            case.update(B=_log_int(rng, 1, 64), S=_length(rng, 16, 16384), causal=rng.random() < 0.5)
            group = rng.choice([1, 1, 4, 8]) if kind == "bwd" else 1
            hkv = _log_int(rng, 1, 32 // group)
            case.update(H=hkv * group)
            if kind == "bwd":
                case.update(Hkv=hkv)
            else:
                case.update(lse=rng.random() < 0.5)
                if case["dtype"] == "f16" and rng.random() < 0.25:
                    case.update(qk_std=math.sqrt(2.0))
        else:
            group = rng.choice([1, 4, 8])
            hkv = _log_int(rng, 1, 32 // group)
            case.update(B=_log_int(rng, 1, 64), H=hkv * group, Hkv=hkv, Skv=_length(rng, 64, 65536),
                        fill=rng.choice([1.0, 0.5, 0.1]))
            if rng.random() < 0.65:                       # a decoding step, now and then of a few speculated tokens
                case.update(Sq=rng.choice([1, 1, 1, 4]), causal=True)
            else:                                         # a prefill chunk
                case.update(Sq=min(_length(rng, 32, 2048), max(1, int(case["Skv"] * case["fill"]))), causal=True)
            if kind == "paged":
                case.update(block_rows=rng.choice([64, 128, 256]))
        w = work(case)
        if w["flops"] <= MOST_FLOPS and w["bytes"] <= MOST_BYTES:
            return case


def _lengths(case):
    """Valid key rows of each batch entry: spread evenly from fill * Skv to Skv."""
    B, Skv, fill = case["B"], case["Skv"], case["fill"]
    if fill == 1.0:
        return [Skv] * B
    return [max(1, int(Skv * (fill + (1.0 - fill) * (b + 0.5) / B))) for b in range(B)]


def prepare(case, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    dtype = DTYPES[case["dtype"]]

    def normal(*shape, std=1.0):
        x = torch.randn(shape, dtype=torch.float32, device="cuda", generator=g)
        return (x if std == 1.0 else x * std).to(dtype)

    B, H, D = case["B"], case["H"], case["D"]
    state = dict(kind=case["kind"], causal=case["causal"])
    if case["kind"] == "fwd":
        S, std = case["S"], case.get("qk_std", 1.0)
        state.update(q=normal(B, H, S, D, std=std), k=normal(B, H, S, D, std=std), v=normal(B, H, S, D), lse=case["lse"])
    elif case["kind"] == "bwd":
        S, Hkv = case["S"], case["Hkv"]
        q, k, v = normal(B, H, S, D), normal(B, Hkv, S, D), normal(B, Hkv, S, D)
        # what the forward pass of the training step left: its output and log-sum-exp
        forward = lib.sdpa if Hkv == H else lib.sdpa_kv
        o, lse = forward(q, k, v, case["causal"], return_lse=True)
        state.update(q=q, k=k, v=v, o=o, lse=lse, dout=normal(B, H, S, D))
    else:
        Hkv, Sq, Skv = case["Hkv"], case["Sq"], case["Skv"]
        order = torch.randperm(B, device="cuda", generator=g)
        lens = torch.tensor(_lengths(case), dtype=torch.int32, device="cuda")[order].contiguous()
        state.update(q=normal(B, H, Sq, D))
        if case["kind"] == "kv":
            state.update(k=normal(B, Hkv, Skv, D), v=normal(B, Hkv, Skv, D), lens=None if case["fill"] == 1.0 else lens)
        else:
            rows = case["block_rows"]
            blocks = -(-Skv // rows)
            pages = torch.randperm(B * blocks, device="cuda", generator=g).to(torch.int32)     # in no order, as a pool hands them out
            state.update(k=normal(B * blocks, Hkv, rows, D), v=normal(B * blocks, Hkv, rows, D), lens=lens,
                         table=pages.view(B, blocks).contiguous())
    return state


def run(state):
    s = state
    if s["kind"] == "fwd":
        return lib.sdpa(s["q"], s["k"], s["v"], s["causal"], return_lse=s["lse"])
    if s["kind"] == "kv":
        return lib.sdpa_kv(s["q"], s["k"], s["v"], s["causal"], kv_lens=s["lens"])
    if s["kind"] == "paged":
        return lib.sdpa_paged(s["q"], s["k"], s["v"], s["lens"], s["table"], s["causal"])
    return lib.sdpa_backward(s["q"], s["k"], s["v"], s["o"], s["dout"], s["lse"], s["causal"])


def work(case):
    B, H, D = case["B"], case["H"], case["D"]
    if case["kind"] in ("fwd", "bwd"):
        S, Hkv = case["S"], case.get("Hkv", H)
        pairs = B * H * (S * (S + 1) // 2 if case["causal"] else S * S)
        if case["kind"] == "fwd":
            return {"bytes": 2 * B * S * D * (2 * H + 2 * Hkv) + (4 * B * H * S if case["lse"] else 0), "flops": 4 * D * pairs}
        # q, o, dout in and dq out; k, v in and dk, dv out; the log-sum-exp in
        return {"bytes": 2 * B * S * D * (4 * H + 4 * Hkv) + 4 * B * H * S, "flops": 10 * D * pairs}
    Sq, lens = case["Sq"], _lengths(case)
    pairs = 0
    for n in lens:
        # under the causal mask query i of the last Sq positions sees n - Sq + i + 1 keys
        pairs += sum(max(0, n - Sq + i + 1) for i in range(Sq)) if case["causal"] else n * Sq
    return {"bytes": 2 * D * (2 * case["Hkv"] * sum(lens) + 2 * B * H * Sq), "flops": 4 * D * H * pairs}


def tolerance(case):
    # Outputs and gradients: 2-norm error against the same path in 64 bits, over the listed and a dozen drawn cases,
    # 1.7e-3 to 2.5e-3 in BF16 and 2.1e-4 to 3.5e-4 in FP16 (P and dS are rounded to 16 bits before the second
    # products, results once more).  About four times that.
    return {"rel": 1e-2 if case["dtype"] == "bf16" else 1.3e-3}
