"""What a serving program has this library do, as cases that can be timed and compared.

A case is one attention layer's shape, format and context, and one of these kinds of pass:

  step      one decode step: for every layer, skvq_append_decode_attention on that layer's own cache
            (long contexts; a pass adds a token to each cache)
  generate  a short request: skvq_prefill_quantize of the prompt into every layer's cache, then a few
            decode steps over the layers (short contexts; every pass starts over)
  verify    skvq_decode_attention_multi: several query tokens per sequence over a long cache, as when
            speculated tokens are checked
  prefill   skvq_prefill_attention_quantize: the whole prefill phase of one layer
  quantize  skvq_prefill_quantize of a prompt, its attention computed elsewhere

Inputs follow the synthetic recipe of paper_2405_06219_amd.synth: normal values with a channel
magnitude profile spread over two decades, channels reordered by their range, clip scale 0.95,
window 128.  Layers rotate so that a pass does not find its data in the 256 MB last-level cache
where a model's many layers would have displaced it.
"""
from __future__ import annotations

import math

import torch

from paper_2405_06219_amd import binding, synth

D = 128
WINDOW = 128
HEADROOM = 16384     # tokens that "step" passes may append to a state
META_BYTES = {"f32": 4, "f16": 2, "e4m3": 1}
CODE_BYTES_K = {2.0: 32, 3.0: 48, 4.0: 64}              # per (token, kv head)
CODE_BYTES_V = {1.5: 26, 2.0: 32, 3.0: 48, 4.0: 64}
BOUNDS = {64: (0, 32, 128), 32: (0, 16, 32, 64, 128)}   # unequal groups: clusters of these sizes


def _case(name, kind, batch, q_heads, kv_heads, context, k_bits=2.0, v_bits=1.5, group=128, meta="f32", sinks=0,
          unequal=False, layers=1, steps=0, new_tokens=1):
    return {"name": name, "kind": kind, "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads, "context": context,
            "k_bits": k_bits, "v_bits": v_bits, "group": group, "meta": meta, "sinks": sinks, "unequal": unequal,
            "layers": layers, "steps": steps, "new_tokens": new_tokens}


def listed():
    return [
        # the smallest calls: a small model's chat turn, 2k tokens of context; launches and latency count
        _case("generate_4heads_2k", "generate", 1, 4, 4, 2048, v_bits=2.0, layers=4, steps=8),
        # ordinary batched serving of a grouped-query model at a few thousand tokens of context, in the
        # paper's 4-bit setting (groups of 64, FP8 scale and zero, five attention sinks)
        _case("generate_batch8_6k_4bit", "generate", 8, 32, 8, 6007, k_bits=4.0, v_bits=4.0, group=64, meta="e4m3",
              sinks=5, layers=6, steps=8),
        # one long document: the decode step at 32k tokens with a head per query head
        _case("step_32heads_32k", "step", 1, 32, 32, 32768, layers=8),
        # the headline: the decode step of a grouped-query model at 128k tokens
        _case("step_gqa_128k", "step", 1, 32, 8, 131072, layers=8),
        # the same model in the paper's accuracy setting: groups of 64, FP8 scale and zero, sinks; odd length
        _case("step_gqa_100k_g64_e4m3", "step", 1, 32, 8, 100003, group=64, meta="e4m3", sinks=5, layers=8),
        # the largest decode calls: one sequence of a million tokens, and a batch of long ones
        _case("step_32heads_1m", "step", 1, 32, 32, 1048576),
        _case("step_batch16_32k", "step", 16, 32, 32, 32768),
        # four speculated tokens checked at once
        _case("verify4_gqa_128k", "verify", 1, 32, 8, 131072, layers=8, new_tokens=4),
        # the prefill phase: a long prompt, and a batch of ordinary ones of odd length
        _case("prefill_gqa_32k", "prefill", 1, 32, 8, 32768),
        _case("prefill_batch2_1913", "prefill", 2, 32, 32, 1913),
        # quantizing a prompt: the headline's, and 3-bit codes in unequal groups at an odd length
        _case("quantize_gqa_128k", "quantize", 1, 32, 8, 131072),
        _case("quantize_batch2_20k_3bit_unequal", "quantize", 2, 32, 32, 20011, k_bits=3.0, v_bits=3.0, group=64,
              meta="e4m3", sinks=5, unequal=True),
    ]


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def _layers_for(case):
    """Layers whose packed data exceeds the last-level cache, at most eight."""
    return max(1, min(8, -(-500_000_000 // max(_packed_bytes(case), 1))))


def draw(rng):
    """One more case: any of the heads, code widths, group sizes and formats of the tests, contexts over
    the range of the listed cases for its kind, no more work than the largest of them."""
    kind = rng.choice(["generate", "generate", "step", "step", "step", "verify", "prefill", "quantize"])
    q_heads, kv_heads = rng.choice([(4, 4), (8, 1), (8, 8), (16, 4), (24, 8), (32, 8), (32, 32)])
    k_bits, v_bits = rng.choice([(2.0, 1.5), (2.0, 1.5), (2.0, 1.5), (2.0, 2.0), (2.0, 4.0), (3.0, 3.0), (4.0, 4.0)])
    group, meta, unequal = rng.choice([(128, "f32", False), (128, "f32", False), (128, "e4m3", False), (64, "e4m3", False),
                                       (64, "f16", True), (32, "e4m3", False)])
    sinks = rng.choice([0, 5])
    # largest (sequence, kv head, token) count of the kind: that of the listed cases
    low, high, most = {"generate": (500, 16384, 3_000_000), "step": (32768, 1048576, 33_000_000),
                       "verify": (4096, 131072, 4_000_000), "prefill": (300, 32768, 0),
                       "quantize": (2000, 131072, 2_000_000)}[kind]
    context = _log_int(rng, low, high)
    if kind == "prefill":  # the score products of the 32k-token prompt
        fits = 32 * 32768 * 32768 // (q_heads * context * context)
    else:
        fits = most // (kv_heads * context)
    if fits < 1:
        context = int(context * fits) if fits else max(low, most // kv_heads)
        fits = 1
    batch = _log_int(rng, 1, max(1, min(16, fits)))
    case = _case("", kind, batch, q_heads, kv_heads, context, k_bits, v_bits, group, meta, sinks, unequal,
                 steps=rng.choice([4, 8]) if kind == "generate" else 0,
                 new_tokens=rng.choice([2, 3, 4, 8]) if kind == "verify" else 1)
    case["layers"] = min(4, _layers_for(case)) if kind == "generate" else 1 if kind == "prefill" else _layers_for(case)
    if kind == "quantize":
        case["layers"] = min(4, case["layers"])
    del case["name"]
    return case


def _workload(case, seed):
    return synth.Workload("case", case["batch"], case["q_heads"], case["kv_heads"], case["context"], case["v_bits"],
                          group_size=case["group"], window=WINDOW, seed=1 + seed % 1_000_003, k_bits=case["k_bits"])


def prepare(case, seed):
    """The layers' caches (prefilled for "step" and "verify"), the prompt where the pass takes it in, the
    queries and new tokens, and the output buffers."""
    device = torch.device("cuda:0")
    w = _workload(case, seed)
    kind, layers = case["kind"], case["layers"]
    b, hq, hk, T = case["batch"], case["q_heads"], case["kv_heads"], case["context"]
    sk, sv = (torch.from_numpy(s).to(device)[None, :, :] for s in synth.channel_scales(w))
    ck, cv = synth.make_clip(w)
    gen = torch.Generator(device=device)
    gen.manual_seed(w.seed)
    room = HEADROOM if kind == "step" else case["steps"]
    tcap = -(-(max(T - WINDOW, 1) + room) // 64) * 64
    state = {"case": case, "caches": [], "prompts": []}
    for layer in range(layers):
        k, v, pk, pv = synth.make_kv_device(w, device, stream=layer)
        cache = binding.SkvqCache(b, hq, hk, case["group"], case["v_bits"], WINDOW, tcap, pk, pv, ck, cv,
                                  k_bits=case["k_bits"], device=device, fill=0, n_sink=case["sinks"], meta=case["meta"],
                                  group_bounds=BOUNDS[case["group"]] if case["unequal"] else None,
                                  max_new_tokens=case["new_tokens"])
        if kind in ("step", "verify"):
            cache.skvq_prefill_quantize(k, v)
        else:
            state["prompts"].append((k, v))
        del k, v
        state["caches"].append(cache)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=device)

    if kind == "prefill":
        state["q"] = normal(b, hq, T, D).to(torch.float16)
        state["out"] = torch.empty((b, hq, T, D), dtype=torch.float32, device=device)
    elif kind in ("step", "generate", "verify"):
        n = max(case["steps"], 1)
        new = (case["new_tokens"],) if kind == "verify" else ()
        q = normal(n, layers, b, *new, hq, D).to(torch.float16)
        kn = (normal(n, layers, b, hk, D) * sk).to(torch.float16)
        vn = (normal(n, layers, b, hk, D) * sv).to(torch.float16)
        state["out"] = torch.empty(q.shape, dtype=torch.float32, device=device)
        # the tensors of every call, as a program's own loop would hold them
        state["q"], state["kn"], state["vn"], state["outs"] = (
            [[t[s][i] for i in range(layers)] for s in range(n)] for t in (q, kn, vn, state["out"]))
    return state


def _buffers(state):
    return [[c.buffers[n] for n in ("k_codes", "v_codes", "k_meta", "v_meta", "k_win", "v_win")] for c in state["caches"]]


def run(state):
    """One pass.  Returns the attention outputs and, where the pass changes them, the caches' buffers."""
    kind, caches = state["case"]["kind"], state["caches"]
    if kind == "prefill":
        caches[0].skvq_prefill_attention_quantize(state["q"], *state["prompts"][0], out_f32=state["out"])
        return state["out"], _buffers(state)
    if kind == "quantize":
        for c, (k, v) in zip(caches, state["prompts"]):
            c.skvq_prefill_quantize(k, v)
        return _buffers(state)
    if kind == "verify":
        for c, q, o in zip(caches, state["q"][0], state["outs"][0]):
            c.skvq_decode_attention_multi(q, out_f32=o)
        return state["out"]
    if kind == "generate":
        for c, (k, v) in zip(caches, state["prompts"]):
            c.skvq_prefill_quantize(k, v)
    for step in range(len(state["q"])):
        for c, q, kn, vn, o in zip(caches, state["q"][step], state["kn"][step], state["vn"][step], state["outs"][step]):
            c.skvq_append_decode_attention(kn, vn, q, out_f32=o)
    return state["out"], _buffers(state)


def _row_bytes(case):
    return (CODE_BYTES_K[case["k_bits"]] + CODE_BYTES_V[case["v_bits"]]
            + 4 * META_BYTES[case["meta"]] * (D // case["group"]))


def _packed_bytes(case):
    return case["batch"] * case["kv_heads"] * max(case["context"] - WINDOW - case["sinks"], 0) * _row_bytes(case)


def _decode_bytes(case, queries):
    """Packed rows and fp16 rows read once, the queries read, the fp32 outputs written."""
    fp16_rows = min(case["context"], WINDOW + case["sinks"])
    return (_packed_bytes(case) + case["batch"] * case["kv_heads"] * fp16_rows * 4 * D
            + case["batch"] * queries * case["q_heads"] * D * 6)


def _quantize_bytes(case):
    """The prompt's K and V read, packed rows and fp16 rows written."""
    rows = case["batch"] * case["kv_heads"]
    return rows * (case["context"] + min(case["context"], WINDOW + case["sinks"])) * 4 * D + _packed_bytes(case)


def work(case):
    b, hq, T, layers = case["batch"], case["q_heads"], case["context"], case["layers"]
    pair = 4 * D  # flops of one (query, token) pair: score and weighted value
    if case["kind"] == "prefill":
        return {"bytes": _quantize_bytes(case) + b * hq * T * D * 6, "flops": b * hq * (T * (T + 1) // 2) * pair}
    if case["kind"] == "quantize":
        return {"bytes": layers * _quantize_bytes(case), "flops": 0}
    if case["kind"] == "generate":
        n = layers * case["steps"]
        return {"bytes": layers * _quantize_bytes(case) + n * _decode_bytes(case, 1), "flops": n * b * hq * T * pair}
    n = case["new_tokens"]
    return {"bytes": layers * _decode_bytes(case, n), "flops": layers * n * b * hq * T * pair}


def tolerance(case):
    """Codes, scales and window rows are bytes and equal.  Attention outputs are sums with fp32 accumulation:
    against the same attention in 64 bits the decode outputs are off by 1e-6 (32k tokens) to 1.2e-5 (a million
    tokens: the matrix cores' accumulation) of their norm and at most 2.4e-5 elementwise, the prompt's by 1.7e-6
    and 8e-6; four times that."""
    if case["kind"] == "quantize":
        return "exact"
    if case["kind"] == "prefill":
        return {"rel": 1e-5, "max": 5e-5}
    return {"rel": 5e-5, "max": 2e-4}
