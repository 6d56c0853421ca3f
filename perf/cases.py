"""Timed cases of the chunk-attention path: what a serving or prefill loop has this library do, call by call.

A case is one call of a public entry point (`ChunkBuffers.chunk_attn`, `ChunkBuffers.dense_attn` or
`PrefillBuffers.run`) on buffers that such a program keeps.  Sizes are those of this repository's workloads
(gen/workloads.py), benchmark and tests, or generic ones of the same ranges.

Fields of a case
  op         "chunk": select and attend for one chunk; "dense": attention over the whole cache; "prefill": a whole
             prompt, chunk after chunk
  dtype      "bf16" or "f32"
  batch, n_q, n_kv, d, chunk      sequences, query heads, KV heads, head size, tokens per chunk
  kv_max, kv_min                  cached tokens per sequence: the first one kv_max, the others spread down to kv_min
                                  ("prefill": kv_max is the prompt length)
  n_retain, budget_pct            retained queries; key budget in per cent of each sequence's cache
  keys       "normal": independent keys; "clustered": sixteen clusters per KV head
  scale_f32  QUOKA_ATTN_SCALE_F32, the option for logits well beyond unit variance
"""
import math

import torch

import paper_2602_08722_amd as quoka


def _case(name, op="chunk", dtype="bf16", batch=1, n_q=32, n_kv=8, d=128, chunk=1024, kv_max=8192, kv_min=None,
          n_retain=64, budget_pct=12.0, keys="normal", scale_f32=False):
    case = dict(op=op, dtype=dtype, batch=batch, n_q=n_q, n_kv=n_kv, d=d, chunk=chunk, kv_max=kv_max,
                kv_min=kv_max if kv_min is None else kv_min, n_retain=n_retain, budget_pct=budget_pct, keys=keys,
                scale_f32=scale_f32)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # one generated token after an 8K prompt: the smallest call, all launches and latency
        _case("decode_8k", chunk=1, kv_max=8192),
        # one generated token for eight sequences of mixed length, as a serving batch has them
        _case("decode_batch", batch=8, chunk=1, kv_max=65536, kv_min=4096),
        # the small float32 problem that checks a build (and every caller that keeps float32 tensors)
        _case("f32_small", dtype="f32", n_q=2, n_kv=1, d=64, chunk=128, kv_max=1024, n_retain=16, budget_pct=12.5),
        # a float32 layer of ordinary size
        _case("f32_4k", dtype="f32", n_q=8, n_kv=2, chunk=512, kv_max=4096),
        # a chunk after a short context
        _case("chunk_8k", chunk=1024, kv_max=8192),
        # a chunk after a medium context, clustered keys
        _case("chunk_32k", chunk=2048, kv_max=32768, n_retain=128, keys="clustered"),
        # a long-context chunk: the largest single call
        _case("chunk_128k", chunk=4096, kv_max=131072, n_retain=128, budget_pct=6.25),
        # short chunks of eight sequences of mixed length
        _case("chunk_batch", batch=8, chunk=512, kv_max=64077, kv_min=4096),
        # nothing divides anything: three heads a group, a ragged chunk, small heads, scale applied in float32
        _case("chunk_odd", batch=3, n_q=12, n_kv=4, d=64, chunk=333, kv_max=19999, kv_min=1237, n_retain=48,
              budget_pct=25.0, scale_f32=True),
        # speculative or multi-token decoding over a long context: a few tokens at once
        _case("tokens_100k", chunk=5, kv_max=100003, n_retain=32, budget_pct=4.0),
        # attention over the whole cache, what the sparse path is compared with
        _case("dense_8k", op="dense", chunk=1024, kv_max=8192),
        # a whole prompt in chunks of 1024, the last one short
        _case("prefill_16k", op="prefill", chunk=1024, kv_max=16000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    largest = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["decode", "decode", "f32", "chunk", "chunk", "chunk", "chunk", "dense", "prefill"])
        d = rng.choice([64, 128, 128])
        n_kv, g = rng.choice([(8, 4), (8, 4), (4, 8), (4, 3), (2, 7), (1, 16), (8, 1)])
        n_retain = rng.choice([16, 32, 48, 64, 64, 100, 128])
        pct = rng.choice([4.0, 8.0, 12.0, 12.0, 17.0, 25.0])
        batch = rng.choice([1, 1, 1, 2, 3, 8, 13])
        keys = rng.choice(["normal", "clustered"])
        scale = rng.random() < 0.2
        if kind == "decode":
            kv = _log_int(rng, 1024, 131072)
            c = _case("", op=rng.choice(["chunk", "chunk", "chunk", "dense"]), batch=batch, n_q=n_kv * g, n_kv=n_kv,
                      d=d, chunk=rng.choice([1, 1, 1, 2, 5, 8]), kv_max=kv, kv_min=max(512, kv // rng.choice([1, 2, 8])),
                      n_retain=n_retain, budget_pct=pct, keys=keys)
        elif kind == "f32":
            kv = _log_int(rng, 512, 8192)
            c = _case("", dtype="f32", batch=rng.choice([1, 1, 2]), n_q=2 * rng.choice([1, 2, 4]), n_kv=2, d=d,
                      chunk=_log_int(rng, 32, 700), kv_max=kv, kv_min=max(200, kv // 2), n_retain=rng.choice([16, 48, 64]),
                      budget_pct=pct, keys=keys)
        elif kind == "prefill":
            c = _case("", op="prefill", n_q=n_kv * g, n_kv=n_kv, d=d, chunk=rng.choice([500, 1024, 1024, 2048]),
                      kv_max=_log_int(rng, 3000, 40000), n_retain=n_retain, budget_pct=pct, keys=keys, scale_f32=scale)
        else:
            kv = _log_int(rng, 1024, 131072)
            c = _case("", op=kind, batch=batch, n_q=n_kv * g, n_kv=n_kv, d=d, chunk=_log_int(rng, 64, 4096), kv_max=kv,
                      kv_min=max(512, kv // rng.choice([1, 2, 8])), n_retain=n_retain, budget_pct=pct, keys=keys,
                      scale_f32=scale)
        if 2 * c["batch"] * c["n_kv"] * c["kv_max"] * c["d"] <= 1 << 29 and _cost(c) <= largest:
            return c


def _lens(case):
    """Cached tokens of every sequence: kv_max first, the others spread over [kv_min, kv_max] without order."""
    lo, hi = case["kv_min"], case["kv_max"]
    return [hi - int((hi - lo) * ((i * 0.6180339887) % 1.0)) for i in range(case["batch"])]


def _budgets(case, lens):
    return [int(case["budget_pct"] * t / 100.0) for t in lens]


def _flags(case):
    return quoka.QUOKA_ATTN_SCALE_F32 if case["scale_f32"] else 0


def prepare(case, seed):
    """Tensors on the GPU and the buffers a caller keeps.  Queries lean towards one direction per head and a tenth of
    them do not (the queries the method keeps); keys and values have unit variance."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(int(seed))
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    b, n_q, n_kv, d, C, T = (case[k] for k in ("batch", "n_q", "n_kv", "d", "chunk", "kv_max"))
    rows = T if case["op"] == "prefill" else C

    def normal(*shape):
        return torch.randn(*shape, device=dev, generator=gen)

    lean = normal(b, n_q, 1, d)
    lean = lean / lean.norm(dim=-1, keepdim=True)
    away = (torch.rand(b, n_q, rows, 1, device=dev, generator=gen) < 0.1).float()
    q = normal(b, n_q, rows, d)
    q = (q + (1.5 * (1.0 - away) - away * (q * lean).sum(-1, keepdim=True)) * lean).to(dt)

    centres = normal(b, n_kv, 16, d)

    def make_keys(n):
        if case["keys"] == "normal":
            return normal(b, n_kv, n, d).to(dt)
        z = torch.randint(0, 16, (b, n_kv, n, 1), device=dev, generator=gen).expand(b, n_kv, n, d)
        return (torch.gather(centres, 2, z) + 0.5 * normal(b, n_kv, n, d)).to(dt)

    k, v = make_keys(T), normal(b, n_kv, T, d).to(dt)
    if case["op"] == "prefill":
        return {"op": "prefill",
                "buf": quoka.PrefillBuffers(q, k, v, C, case["n_retain"],
                                            lambda t: int(case["budget_pct"] * t / 100.0), score_flags=_flags(case))}
    lens = _lens(case)
    buf = quoka.ChunkBuffers(q, k, v, make_keys(C), normal(b, n_kv, C, d).to(dt), lens, _budgets(case, lens),
                             case["n_retain"], score_flags=_flags(case))
    buf.k_idx.zero_()   # lists of short sequences end before the array does
    return {"op": case["op"], "buf": buf}


def run(state):
    buf = state["buf"]
    if state["op"] == "prefill":
        return {"out": buf.run(sparse=True)}
    if state["op"] == "dense":
        return {"out": buf.dense_attn(), "lse": buf.lse}
    return {"out": buf.chunk_attn(), "lse": buf.lse, "k_idx": buf.k_idx, "k_cnt": buf.k_cnt}


def work(case):
    """What one pass cannot do without.  Sparse: Q once, every cached key once (scoring), the selected keys' values and
    the chunk's own keys and values once, the output and the index lists once; products of the retained queries with
    the cache and of every query with what it attends."""
    es = 2 if case["dtype"] == "bf16" else 4
    n_q, n_kv, d = case["n_q"], case["n_kv"], case["d"]
    total = {"bytes": 0.0, "flops": 0.0}

    def chunk(T, C, sparse):
        n_keep = min(case["n_retain"], C)
        B = min(int(case["budget_pct"] * T / 100.0), T) if sparse else T
        total["bytes"] += 2.0 * n_q * C * d * es + 2.0 * n_kv * C * d * es + float(n_kv) * (T + B) * d * es
        total["flops"] += 4.0 * n_q * d * (C * B + C * (C + 1) / 2.0)
        if sparse:
            total["bytes"] += 4.0 * n_kv * B
            total["flops"] += 2.0 * n_kv * n_keep * T * d

    if case["op"] == "prefill":
        for t in range(0, case["kv_max"], case["chunk"]):
            chunk(t, min(case["chunk"], case["kv_max"] - t), True)
    else:
        for t in _lens(case):
            chunk(t, case["chunk"], case["op"] == "chunk")
    return total


def _cost(case):
    w = work(case)
    peak = 2.5e15 if case["dtype"] == "bf16" else 1.5e14
    return max(w["bytes"] / 8e12, w["flops"] / peak)


def tolerance(case):
    """Measured against attention in float64 over the same key lists: 6e-7 (float32; largest difference 7e-6 of the
    output's root mean square), 2.9e-3 (bf16: the queries, the probabilities and the output are each rounded once;
    largest difference 0.04).  Key lists are whole numbers: only scores that tie in the last float32 bits may go either
    way."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 1e-4, "differ": 0.01}
    return {"rel": 1e-2, "max": 0.15, "differ": 0.01}
