"""Timing cases of the cascading KV cache: what a program that serves or streams text through it asks for.

A case is one of four kinds of call sequence on a cache that has been in use for `context` tokens:

  decode   one token for every sequence of the batch, through `layers` layers
  chunk    one chunk of strided prefill (steady state of a long prompt)
  turn     a user turn of a conversation: the prompt of `chunk` tokens, `steps` generated tokens, and the
           host's view of what the cache holds (read_state) for the session store
  prompt   a whole new request: a cache is opened, `context` tokens are fed in chunks, the cache is closed

Ring heads, acceptance phases and fills are those of a stream of that length: the structure of the cache
follows from the token count (cascade_simulate_structure), its rows and scores are drawn, and a few calls
are made before the first timed one, so that the rings are turned and whatever a cache keeps from call to call is
in its usual state.  Keys, values and queries are N(0,1), as in the package's workloads.
"""
import math

import torch

from paper_2406_17808_amd import binding as B
from paper_2406_17808_amd.cache import CascadeKVCache, CascadeKVLayers

DEVICE = "cuda:0"

BASE = dict(kind="chunk", dtype="bf16", batch=1, hq=32, hkv=8, d=128, sinks=64, cascades=4, size=4096, context=1 << 18, chunk=4096,
            max_chunk=4096, steps=0, layers=1, beta=0.9999, base=500000.0, scale=1.0, single_pass=False, homogeneous=False, mean=False)


def listed():
    def case(name, **over):
        return dict(BASE, name=name, **over)

    return [
        # interactive generation, one conversation, one layer: latency and launches
        case("decode_b1_8k", kind="decode", size=2048, chunk=1, max_chunk=512, steps=1),
        # the same through all layers of a model of the 8B class that share one scratch
        case("decode_layers32_4k", kind="decode", size=1024, chunk=1, max_chunk=1024, steps=1, layers=32, beta=0.9),
        # a middling batch of decoders on the cache of the paper's latency figure
        case("decode_b8_16k", kind="decode", batch=8, chunk=1, max_chunk=512, steps=1),
        # the largest decode workload: 32 sequences, 65K slots each, bound by memory
        case("decode_b32_65k", kind="decode", batch=32, size=16384, context=1 << 20, chunk=1, max_chunk=1, steps=1, beta=0.9),
        # the fp32 configuration: one head, chunks of 32
        case("chunk32_f32", dtype="f32", hq=1, hkv=1, d=64, sinks=4, size=64, context=1024, chunk=32, max_chunk=32, beta=0.9, base=10000.0),
        # a whole request of the long-context-understanding experiment: 40000 tokens, stride 512, ragged last chunk
        case("prompt_40000_8k", kind="prompt", size=2048, context=40000, chunk=512, max_chunk=512),
        # short chunks on a small cache, few rows in the scores, small logits
        case("chunk1024_4k", size=1024, context=32768, chunk=1024, max_chunk=1024, beta=0.9, scale=1.0 / math.sqrt(128.0)),
        # eight cascades: many segments
        case("chunk2048_16k_c8", cascades=8, size=2048, context=131072, chunk=2048, max_chunk=2048, beta=0.9),
        # the paper's latency figure: every row of a chunk carries weight in the scores
        case("chunk4096_16k"),
        # the same with the scores taken inside the attention sweep
        case("chunk4096_16k_single_pass", single_pass=True),
        # the headline workload: 1M tokens against 65K slots
        case("chunk4096_65k", size=16384, context=1 << 19, beta=0.9),
        # a turn of two conversations: head size 64, eight query heads per KV head, ragged lengths, prefill and decode mixed
        case("turn_b2_3k_d64", kind="turn", batch=2, hq=16, hkv=2, d=64, sinks=32, cascades=3, size=1024, context=16000, chunk=300,
             max_chunk=512, steps=8, beta=0.99),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    largest = [work(c) for c in listed()]
    top_flops, top_bytes = max(w["flops"] for w in largest), max(w["bytes"] for w in largest)
    while True:
        c = dict(BASE)
        c["kind"] = rng.choices(["decode", "chunk", "turn", "prompt"], [4, 5, 2, 1])[0]
        c["dtype"] = rng.choices(["bf16", "f32"], [7, 1])[0]
        c["d"] = rng.choice([64, 128, 128])
        c["hkv"] = rng.choice([1, 2, 4, 8, 8])
        c["hq"] = c["hkv"] * rng.choice([1, 2, 4, 4, 5, 8])
        c["cascades"] = rng.choice([1, 2, 3, 4, 4, 8])
        c["sinks"] = rng.choice([4, 64, 64, rng.randrange(0, 65)])
        total = _log_int(rng, 512, 65536)
        # sizes of whole tiles as in the experiments, and odd ones
        c["size"] = max(16, total // c["cascades"] // 64 * 64) if rng.random() < 0.6 else max(16, total // c["cascades"])
        slots = c["sinks"] + c["cascades"] * c["size"]
        c["beta"] = rng.choice([0.9, 0.99, 0.9999, 0.9999])
        c["homogeneous"] = rng.random() < 0.15
        c["mean"] = rng.random() < 0.15
        c["base"] = rng.choice([10000.0, 500000.0])
        # mostly caches that a long stream has filled, some that are still filling
        c["context"] = min(c["size"] << c["cascades"], 1 << 20) if rng.random() < 0.7 else _log_int(rng, 256, 16 * slots)
        chunk = _log_int(rng, 16, 4096)
        if rng.random() < 0.6:
            chunk = max(16, 1 << int(math.log2(chunk) + 0.5))
        if c["kind"] == "decode":
            c["batch"], c["chunk"], c["steps"] = _log_int(rng, 1, 32), 1, 1
            c["max_chunk"] = rng.choice([1, 512])
            c["layers"] = rng.choice([1, 1, 2, 16]) if slots <= 8300 and c["batch"] <= 4 else 1
        else:
            c["batch"] = rng.choice([1, 1, 1, 2, 3]) if c["kind"] != "prompt" else 1
            c["chunk"] = c["max_chunk"] = chunk
            if c["kind"] == "turn":
                c["steps"] = rng.randrange(1, 9)
                c["max_chunk"] = chunk + rng.randrange(0, 200)
            if c["kind"] == "prompt":
                c["context"] = _log_int(rng, 256, 32768)
            c["single_pass"] = c["dtype"] == "bf16" and c["beta"] > 0.999 and rng.random() < 0.3
        if c["dtype"] == "f32" and (slots > 4200 or c["chunk"] > 256 or c["batch"] > 2 or c["hq"] > 16 or c["kind"] == "prompt"):
            continue      # fp32 is there for small, exact work
        w = work(c)
        if w["flops"] <= top_flops and w["bytes"] <= top_bytes and c["context"] / c["chunk"] < (400 if c["kind"] == "prompt" else 1e9):
            return c


def _config(c):
    return B.make_config(batch=c["batch"], n_q_heads=c["hq"], n_kv_heads=c["hkv"], head_dim=c["d"],
                         dtype=B.CASCADE_BF16 if c["dtype"] == "bf16" else B.CASCADE_F32, n_sink=c["sinks"],
                         cascade_sizes=[c["size"]] * c["cascades"], ema_beta=c["beta"], rope_base=c["base"], max_chunk=c["max_chunk"],
                         head_reduce=B.CASCADE_REDUCE_MEAN if c["mean"] else B.CASCADE_REDUCE_MAX,
                         head_policy=B.CASCADE_HEADS_HOMOGENEOUS if c["homogeneous"] else B.CASCADE_HEADS_INDEPENDENT,
                         score_mode=B.CASCADE_SCORES_SINGLE_PASS if c["single_pass"] else B.CASCADE_SCORES_EXACT)


def _torch_dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _normal(c, gen, shape):
    x = torch.randn(shape, generator=gen, device=DEVICE, dtype=_torch_dtype(c))
    return x if c["scale"] == 1.0 else x * c["scale"]


def _used_cache(c, cfg, gen):
    """The initial state of one layer after `context` tokens, and the tensors it points to."""
    st = B.cascade_simulate_structure(cfg, [c["context"]])
    counts = [int(x) for x in st.counts]
    n = sum(counts)
    shape = (c["batch"], c["hkv"], n)
    k, v = _normal(c, gen, shape + (c["d"],)), _normal(c, gen, shape + (c["d"],))
    mu = torch.rand(shape, generator=gen, device=DEVICE, dtype=torch.float32) / max(n, 1)
    if c["homogeneous"]:      # one score per token for all heads
        mu = mu[:, :1].expand(shape).contiguous()
    ids = torch.cat([torch.arange(counts[0]), torch.arange(c["context"] - (n - counts[0]), c["context"])])
    ids = ids.to(torch.int32).to(DEVICE).expand(shape).contiguous()
    init = B.cascade_init_state()
    init.dev_k, init.dev_v, init.dev_mu, init.dev_ids = k.data_ptr(), v.data_ptr(), mu.data_ptr(), ids.data_ptr()
    for i, x in enumerate(counts):
        init.counts[i] = x
    init.t, init.n_seen = int(st.t), int(st.n_seen)
    return init, (k, v, mu, ids)


def _chunk_inputs(c, gen, n):
    b, d = c["batch"], c["d"]
    return tuple(_normal(c, gen, (b, n, h, d)) for h in (c["hq"], c["hkv"], c["hkv"]))


def _step_inputs(c, gen):
    b, d = c["batch"], c["d"]
    return tuple(_normal(c, gen, (b, h, d)) for h in (c["hq"], c["hkv"], c["hkv"]))


def prepare(case, seed):
    c = dict(BASE, **case)
    cfg = _config(c)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    state = {"case": c, "cfg": cfg, "at": 0}
    if c["kind"] == "prompt":
        state["tokens"] = _chunk_inputs(c, gen, c["context"])
        state["out"] = torch.empty_like(state["tokens"][0])
        return state
    held = [_used_cache(c, cfg, gen) for _ in range(c["layers"])]
    if c["layers"] > 1:
        state["owner"] = CascadeKVLayers(cfg, c["layers"], DEVICE, [h[0] for h in held])
        caches = state["owner"].layers
    else:
        caches = [CascadeKVCache(cfg, DEVICE, held[0][0])]
    state["caches"] = caches
    torch.cuda.synchronize()
    del held
    # tokens to come: taken in turn, so that successive calls bring other tokens
    if c["kind"] != "decode":
        state["chunks"] = [_chunk_inputs(c, gen, c["chunk"]) for _ in range(4)]
        state["chunk_out"] = torch.empty_like(state["chunks"][0][0])
    if c["steps"]:
        state["tokens"] = [_step_inputs(c, gen) for _ in range(max(32, c["steps"]))]
        state["step_outs"] = [[torch.empty_like(state["tokens"][0][0]) for _ in range(c["steps"])] for _ in caches]
    # the stream just before the first pass: ring heads away from slot 0 and off the tile grid
    first = max(1, c["max_chunk"] - c["sinks"]) if c["max_chunk"] > 1 else 0
    for cache in caches:
        if first:
            cache.prefill_chunk(*_chunk_inputs(c, gen, first))
        if c["kind"] == "chunk":
            cache.prefill_chunk(*_chunk_inputs(c, gen, c["chunk"]))
        else:
            for i in range(37 if c["max_chunk"] == 1 else 5):
                cache.decode_step(*state["tokens"][i % 32])
    torch.cuda.synchronize()
    return state


def run(state):
    c = state["case"]
    if c["kind"] == "prompt":
        q, k, v = state["tokens"]
        out = state["out"]
        cache = CascadeKVCache(state["cfg"], DEVICE)
        for a in range(0, c["context"], c["chunk"]):
            b = min(a + c["chunk"], c["context"])
            cache.prefill_chunk(q[:, a:b], k[:, a:b], v[:, a:b], out=out[:, a:b])
        cache.close()
        return out
    at = state["at"]
    state["at"] = at + 1
    outs = []
    if c["kind"] != "decode":
        cache = state["caches"][0]
        outs.append(cache.prefill_chunk(*state["chunks"][at % 4], out=state["chunk_out"]))
    for i in range(c["steps"]):
        token = state["tokens"][(at * c["steps"] + i) % len(state["tokens"])]
        for cache, bufs in zip(state["caches"], state["step_outs"]):
            outs.append(cache.decode_step(*token, out=bufs[i]))
    if c["kind"] == "turn":
        view = state["caches"][0].read_state()
        outs += [view.ids, view.mu, view.slot]
    return outs


def work(case):
    """What a pass cannot do without: every cached key, value and score read once, scores, outputs and new rows written once,
    and the products of queries with the visible keys and of probabilities with the values."""
    c = dict(BASE, **case)
    slots = c["sinks"] + c["cascades"] * c["size"]
    e = 2 if c["dtype"] == "bf16" else 4
    bh = c["batch"] * c["hkv"]
    row = 2 * c["d"] * e

    def call(n, q):      # q tokens on n cached rows
        nbytes = bh * (n * (row + 8) + q * (2 * row + 8)) + 2 * c["batch"] * q * c["hq"] * c["d"] * e
        flops = 4.0 * c["d"] * c["hq"] * c["batch"] * (q * n + q * (q + 1) / 2)
        return nbytes, flops

    if c["kind"] == "prompt":
        cfg = _config(c)
        calls = []
        seen = 0
        while seen < c["context"]:
            q = min(c["chunk"], c["context"] - seen)
            calls.append(call(B.cascade_simulate_structure(cfg, [seen]).count if seen else 0, q))
            seen += q
    else:
        n = B.cascade_simulate_structure(_config(c), [c["context"]]).count
        calls = [call(n, c["chunk"])] if c["kind"] != "decode" else []
        calls += [call(min(slots, n + c["chunk"]), 1)] * (c["steps"] * c["layers"])
    return {"bytes": float(sum(x[0] for x in calls)), "flops": float(sum(x[1] for x in calls))}


def tolerance(case):
    """bf16: the probabilities are rounded to 8 bits against another maximum when a row's keys are summed in another split, and so
    are the results: 3e-3 measured between splits of the keys, 8e-3 where a selection between two tokens of equal score went
    the other way (another token then sits in that slot).  fp32: sums in another order."""
    if case.get("dtype", "bf16") == "bf16":
        return {"rel": 1.2e-2, "max": 0.3, "differ": 1.5e-3}
    return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
