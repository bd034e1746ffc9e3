"""Cases for timing the library the way a serving program uses it: whole requests through the public binding.

A case names a kind and its sizes:

  steps       a request whose prompt K/V is at hand (a prefix hit, or a prompt prefilled elsewhere): the slots are reset
              and filled, then `tokens` decode steps run through all layers, one pod_decode_step (or
              pod_decode_step_reuse) per layer and token.  `graph`: the request is one captured HIP graph that is replayed.
  gated       one decode attention of every layer over a cache that is already there, with the gated skip of distant
              tokens (half of the kv heads have recent keys that dominate and skip, the others do not).
  prefill     a prompt through all layers of a block, attention and cache construction, then the first decode step.
  chunked     the same with the prompt in chunks, each attending what the cache holds, stored as it goes.
  selection   token selection after a prompt: cache filled, votes, pooled top-k, compaction of all layers, one decode
              attention per layer on what is left.
  similarity  the offline layer similarity of attention rows that the layer grouping reads.

All tensors are N(0,1) in bf16 (keys already rotated, logits scaled by 1/sqrt(head_dim)), as the tests and the benchmark
have them.  `group` layers form a block; `headwise` gives the odd kv heads blocks of half that size.
"""
import math
import random

import torch

import paper_2412_02252_amd as pod

DEV = "cuda:0"

SHAPE_8B = {"q_heads": 32, "kv_heads": 8, "head_dim": 128}


def listed():
    return [
        # a small model (or one shard of it), a short chat, one user: the launches and the latency of each step
        {"name": "step-2k-small", "kind": "steps", "layers": 2, "group": 2, "headwise": False, "q_heads": 4, "kv_heads": 2, "head_dim": 64,
         "sink": 16, "window": 256, "batch": 1, "lo": 2048, "hi": 2048, "tokens": 32, "reuse": False, "graph": True},
        # one user with a long document, the usual model shape
        {"name": "step-32k", "kind": "steps", "layers": 2, "group": 2, "headwise": False, **SHAPE_8B,
         "sink": 64, "window": 2048, "batch": 1, "lo": 32768, "hi": 32768, "tokens": 32, "reuse": False, "graph": True},
        # a server's batch of chats of all lengths with 64-wide heads
        {"name": "step-chats-32", "kind": "steps", "layers": 2, "group": 2, "headwise": False, "q_heads": 16, "kv_heads": 4, "head_dim": 64,
         "sink": 16, "window": 512, "batch": 32, "lo": 300, "hi": 4096, "tokens": 32, "reuse": False, "graph": True},
        # a server's batch of documents of all lengths
        {"name": "step-batch16", "kind": "steps", "layers": 2, "group": 2, "headwise": False, **SHAPE_8B,
         "sink": 64, "window": 2048, "batch": 16, "lo": 4096, "hi": 32768, "tokens": 16, "reuse": False, "graph": False},
        # very long contexts, larger blocks, upper layers on the lowest layer's scores
        {"name": "reuse-128k", "kind": "steps", "layers": 4, "group": 4, "headwise": False, **SHAPE_8B,
         "sink": 128, "window": 4096, "batch": 4, "lo": 131072, "hi": 131072, "tokens": 16, "reuse": True, "graph": False},
        # gated skip with head-wise blocks at a medium batch
        {"name": "gated-24k", "kind": "gated", "layers": 4, "group": 4, "headwise": True, **SHAPE_8B,
         "sink": 64, "window": 2048, "batch": 4, "lo": 16000, "hi": 24000, "tau": 0.9},
        # a question of some hundred tokens
        {"name": "prefill-777", "kind": "prefill", "layers": 2, "group": 2, "headwise": False, **SHAPE_8B,
         "sink": 16, "window": 256, "n": 777},
        # a document of some thousand tokens, 64-wide heads
        {"name": "prefill-3k-d64", "kind": "prefill", "layers": 2, "group": 2, "headwise": False, "q_heads": 16, "kv_heads": 4, "head_dim": 64,
         "sink": 16, "window": 512, "n": 3001},
        # a long document in one call
        {"name": "prefill-16k", "kind": "prefill", "layers": 2, "group": 2, "headwise": False, **SHAPE_8B,
         "sink": 64, "window": 2048, "n": 16384},
        # a document in chunks, as a server does that serves others in between
        {"name": "chunked-8k", "kind": "chunked", "layers": 2, "group": 2, "headwise": False, **SHAPE_8B,
         "sink": 64, "window": 2048, "n": 8192, "chunk": 2048},
        # a long prompt cut down to 4096 stored tokens
        {"name": "selection-16k", "kind": "selection", "layers": 2, "group": 2, "headwise": False, **SHAPE_8B,
         "sink": 64, "window": 2048, "n": 16384, "obs": 64, "keep": 1984, "pool": 7, "pool_max": True},
        # offline: 32 layers, attention rows of sampled queries
        {"name": "similarity-32", "kind": "similarity", "layers": 32, "heads": 32, "rows": 32, "n": 2048},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng):
    return dict(rng.choice([SHAPE_8B, {"q_heads": 16, "kv_heads": 4, "head_dim": 64}, {"q_heads": 16, "kv_heads": 1, "head_dim": 128},
                            {"q_heads": 32, "kv_heads": 4, "head_dim": 128}, {"q_heads": 8, "kv_heads": 8, "head_dim": 64}]))


def draw(rng):
    kind = rng.choice(["steps", "steps", "steps", "gated", "prefill", "prefill", "chunked", "selection", "similarity"])
    if kind == "similarity":
        return {"kind": kind, "layers": rng.randint(8, 32), "heads": rng.choice([4, 8, 16, 32]), "rows": 4 * _log(rng, 1, 8),
                "n": _log(rng, 200, 2048)}
    sink, window = rng.choice([(16, 256), (16, 512), (64, 2048), (4, 1000), (128, 4096)])
    case = {"kind": kind, "layers": 2, "group": 2, "headwise": rng.random() < 0.25, **_shape(rng), "sink": sink, "window": window}
    if rng.random() < 0.3:
        case.update(layers=4, group=4)
    if kind == "steps":
        batch = _log(rng, 1, 48)
        most = max(600, min(65536, 262144 // batch))
        hi = _log(rng, 500, most)
        case.update(batch=batch, lo=max(1, int(hi * rng.choice([1.0, 0.5, 0.1]))), hi=hi, tokens=16, reuse=rng.random() < 0.4,
                    graph=rng.random() < 0.5)
    elif kind == "gated":
        batch = _log(rng, 1, 8)
        case.update(sink=64, window=2048, batch=batch, lo=10000, hi=_log(rng, 10000, 40000), tau=0.9)
    elif kind == "prefill":
        case.update(n=_log(rng, 60, 12000), layers=2, group=2)
    elif kind == "chunked":
        n = _log(rng, 600, 10000)
        case.update(n=n, chunk=min(n, _log(rng, 256, 4096)), layers=2, group=2)
    else:
        n = _log(rng, 4000, 24000)
        case.update(sink=64, window=2048, n=n, obs=rng.choice([16, 32, 64]), keep=rng.randint(200, min(4096, n - 2112)),
                    pool=rng.choice([1, 5, 7]), pool_max=rng.random() < 0.5)
    return case


# ---- what a case means ----

def _lens(case):
    """Stored tokens of each sequence: spread over [lo, hi], the same for every seed."""
    r = random.Random("%(batch)d %(lo)d %(hi)d" % case)
    return [r.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]


def _lowest(case, layer, head):
    g = case["group"]
    if case["headwise"] and head % 2:
        g = max(1, g // 2)
    return layer - layer % g


def _table(case):
    return [[_lowest(case, l, h) for h in range(case["kv_heads"])] for l in range(case["layers"])]


def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.bfloat16)


def _shared(case, per_layer, layer, dim):
    """What an upper layer is given as q_shared / k_shared: each kv head's slice from the lowest layer of its block (None where the
    layer starts every block)."""
    low = _table(case)[layer]
    if all(x == layer for x in low):
        return None
    if len(set(low)) == 1:
        return per_layer[low[0]]
    parts = [t.unflatten(dim, (case["kv_heads"], -1)) for t in per_layer]
    return torch.stack([parts[x].select(dim, h) for h, x in enumerate(low)], dim).flatten(dim, dim + 1).contiguous()


def _cache(case, batch, max_context):
    cfg = pod.make_config(case["layers"], case["group"], case["q_heads"], case["kv_heads"], case["head_dim"], case["sink"],
                          case["window"], batch, max_context, block_lowest=_table(case) if case["headwise"] else None)
    return pod.PodCache(cfg, DEV)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind = case["kind"]
    s = {"case": case, "kind": kind}
    if kind == "similarity":
        a = torch.randn((case["layers"], case["heads"], case["rows"], case["n"]), generator=gen, device=DEV)
        common = torch.randn((1, case["heads"], case["rows"], case["n"]), generator=gen, device=DEV)
        s["att"] = torch.softmax(2.0 * common + a, dim=-1).contiguous()   # layers that resemble one another
        return s
    L, Hq, Hkv, d = case["layers"], case["q_heads"], case["kv_heads"], case["head_dim"]
    s["scale"] = 1.0 / math.sqrt(d)
    if kind in ("steps", "gated"):
        lens = _lens(case)
        B, T = case["batch"], case.get("tokens", 0)
        s["k"] = [[_normal(gen, n, Hkv, d) for n in lens] for _ in range(L)]
        s["v"] = [[_normal(gen, n, Hkv, d) for n in lens] for _ in range(L)]
        s["cache"] = _cache(case, B, max(lens) + T)
        s["scores"] = s["cache"].new_score_buffer() if case.get("reuse") or kind == "gated" else None
        if kind == "gated":
            for layer in range(L):
                for b, n in enumerate(lens):
                    s["k"][layer][b][max(0, n - case["window"]):, 0::2] *= 8.0  # (upper layers' even heads skip)
                    s["cache"].pod_cache_fill(layer, b, s["k"][layer][b], s["v"][layer][b])
            s["q"] = [_normal(gen, B, Hq, d) for _ in range(L)]
            s["ctx"] = torch.tensor(lens, dtype=torch.int32, device=DEV)
            s["out"] = [torch.empty_like(q) for q in s["q"]]
            return s
        s["k_new"] = [[_normal(gen, B, Hkv, d) for _ in range(L)] for _ in range(T)]
        s["v_new"] = [[_normal(gen, B, Hkv, d) for _ in range(L)] for _ in range(T)]
        s["q"] = [[_normal(gen, B, Hq, d) for _ in range(L)] for _ in range(T)]
        s["q_shared"] = [[_shared(case, s["q"][t], l, 1) for l in range(L)] for t in range(T)]
        s["positions"] = [torch.tensor([n + t for n in lens], dtype=torch.int32, device=DEV) for t in range(T)]
        s["out"] = torch.empty((T, L, B, Hq, d), dtype=torch.bfloat16, device=DEV)
        s["graph"] = None
        if case["graph"]:
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                _request(s)
            s["graph"] = g
        return s
    n = case["n"]
    s["q"] = [_normal(gen, n, Hq, d) for _ in range(L)]
    s["k"] = [_normal(gen, n, Hkv, d) for _ in range(L)]
    s["v"] = [_normal(gen, n, Hkv, d) for _ in range(L)]
    s["cache"] = _cache(case, 1, n + 16)
    if kind == "selection":
        s["q"] = [q[n - case["obs"]:].contiguous() for q in s["q"]]
        s["ws"] = s["cache"].new_select_workspace(n, case["obs"], case["keep"])
        # the selection is made from votes that the caller has added up over several observation windows
        s["votes"] = [torch.rand((Hkv, n - case["sink"] - case["window"]), generator=gen, device=DEV) for _ in range(L)]
        s["sel"] = torch.zeros((L, Hkv, case["keep"]), dtype=torch.int32, device=DEV)
        s["fresh"] = [torch.zeros_like(v) for v in s["votes"]]
        s["last"] = [q[-1:].contiguous() for q in s["q"]]
        s["last_shared"] = [_shared(case, s["last"], l, 1) for l in range(L)]
        s["ctx"] = torch.tensor([case["sink"] + case["keep"] + case["window"]], dtype=torch.int32, device=DEV)
        s["out"] = [torch.empty_like(q) for q in s["last"]]
        return s
    s["q_shared"] = [_shared(case, s["q"], l, 1) for l in range(L)]
    s["k_shared"] = [_shared(case, s["k"], l, 1) for l in range(L)]
    s["out"] = [torch.empty_like(q) for q in s["q"]]
    s["k_new"], s["v_new"] = ([_normal(gen, 1, Hkv, d) for _ in range(L)] for _ in range(2))
    s["last"] = [_normal(gen, 1, Hq, d) for _ in range(L)]
    s["last_shared"] = [_shared(case, s["last"], l, 1) for l in range(L)]
    s["positions"] = torch.tensor([n], dtype=torch.int32, device=DEV)
    s["first"] = [torch.empty_like(q) for q in s["last"]]
    if kind == "chunked":
        s["ws"] = s["cache"].new_chunk_workspace(n)
    return s


def _request(s):
    """Reset, fill, then the decode steps of every layer."""
    c, cache, case = s["scale"], s["cache"], s["case"]
    cache.pod_cache_reset()
    for layer in range(case["layers"]):
        for b in range(case["batch"]):
            cache.pod_cache_fill(layer, b, s["k"][layer][b], s["v"][layer][b])
    for t in range(case["tokens"]):
        for layer in range(case["layers"]):
            if case["reuse"]:
                cache.pod_decode_step_reuse(layer, s["k_new"][t][layer], s["v_new"][t][layer], s["q"][t][layer], s["positions"][t], c,
                                            s["scores"], out=s["out"][t, layer])
            else:
                cache.pod_decode_step(layer, s["k_new"][t][layer], s["v_new"][t][layer], s["q"][t][layer], s["q_shared"][t][layer],
                                      s["positions"][t], c, out=s["out"][t, layer])


def run(s):
    kind, case = s["kind"], s["case"]
    if kind == "steps":
        if s["graph"] is not None:
            s["graph"].replay()
        else:
            _request(s)
        return s["out"]
    if kind == "similarity":
        return pod.pod_layer_similarity(s["att"])
    cache, c = s["cache"], s["scale"]
    layers = range(case["layers"])
    if kind == "gated":
        for layer in layers:
            cache.pod_decode_attention_gated(layer, s["q"][layer], s["ctx"], c, case["tau"], s["scores"], out=s["out"][layer])
        return {"out": s["out"], "skipped": cache.skip_flags(s["scores"])}
    cache.pod_cache_reset()
    if kind == "prefill":
        for layer in layers:
            cache.pod_prefill_attention(layer, 0, s["q"][layer], s["k"][layer], s["v"][layer], s["q_shared"][layer], s["k_shared"][layer], c,
                                        out=s["out"][layer], write_cache=True)
    if kind == "chunked":
        for a in range(0, case["n"], case["chunk"]):
            z = slice(a, min(case["n"], a + case["chunk"]))
            for layer in layers:
                qs, ks = s["q_shared"][layer], s["k_shared"][layer]
                cache.pod_prefill_attention_chunk(layer, 0, s["q"][layer][z], s["k"][layer][z], s["v"][layer][z],
                                                  None if qs is None else qs[z], None if ks is None else ks[z], c, s["ws"],
                                                  out=s["out"][layer][z], write_cache=True)
    if kind in ("prefill", "chunked"):
        for layer in layers:
            cache.pod_decode_step(layer, s["k_new"][layer], s["v_new"][layer], s["last"][layer], s["last_shared"][layer], s["positions"], c,
                                  out=s["first"][layer])
        return {"out": s["out"], "first": s["first"]}
    table, n = _table(case), case["n"]
    for layer in layers:
        cache.pod_cache_fill(layer, 0, s["k"][layer], s["v"][layer])
    for layer in layers:
        if layer in table[layer]:
            cache.pod_select_votes(layer, s["q"][layer], s["k"][layer], c, s["ws"], votes=s["fresh"][layer])
            cache.pod_select_top(layer, n, s["votes"][layer], case["pool"], pod.POOL_MAX if case["pool_max"] else pod.POOL_AVG,
                                 case["keep"], s["sel"], s["ws"])
    for layer in layers:
        cache.pod_cache_compact(layer, 0, s["sel"], s["ws"])
    for layer in layers:
        cache.pod_decode_attention(layer, s["last"][layer], s["last_shared"][layer], s["ctx"], c, out=s["out"][layer])
    return {"votes": s["fresh"], "sel": s["sel"], "out": s["out"]}


def work(case):
    """Bytes each call has to read and write once, and the multiply-adds of the products (two operations each)."""
    kind = case["kind"]
    if kind == "similarity":
        L, H, rows, n = case["layers"], case["heads"], case["rows"], case["n"]
        # per pair of layers and element: a sum, a logarithm, a multiply-add
        return {"bytes": 4.0 * L * H * (rows * n + L), "flops": 4.0 * H * rows * n * L * (L - 1) / 2}
    L, Hq, Hkv, d = case["layers"], case["q_heads"], case["kv_heads"], case["head_dim"]
    row, P = 2 * d, case["sink"] + case["window"]
    table = _table(case)
    starts = [sum(x == l for x in table[l]) for l in range(L)]   # kv heads whose block starts at the layer

    def stored(n, low):          # bytes the cache keeps of n tokens at a layer that starts `low` heads' blocks
        dist = max(0, n - P)
        return row * (Hkv * (2 * (n - dist) + dist) + low * dist)

    def fill(n, low):
        return 2 * row * Hkv * n + stored(n, low)

    total = flops = 0.0
    if kind in ("steps", "gated"):
        for n0 in _lens(case):
            for l, low in enumerate(starts):
                if kind == "steps":
                    total += fill(n0, low)
                for n in range(n0 + 1, n0 + 1 + case["tokens"]) if kind == "steps" else [n0]:
                    dist = max(0, n - P)
                    total += row * (2 * Hkv * (n - dist) + Hkv * dist + 2 * Hq)
                    if kind == "steps" and not case["reuse"]:
                        total += row * Hkv * dist
                    else:                      # keys where a block starts, whose logits go out; logits come in elsewhere
                        total += row * low * dist + 4 * Hq * dist
                    if kind == "gated":        # every second head leaves its values and logits out, except where its block starts
                        skip = sum(table[l][h] != l for h in range(0, Hkv, 2))
                        total -= skip * dist * (row + 4 * Hq // Hkv)
                    flops += 4.0 * d * Hq * n
        return {"bytes": total, "flops": flops}
    n = case["n"]
    if kind in ("prefill", "chunked"):
        for low in starts:
            total += row * n * (2 * Hq + 2 * Hkv) + (row * n * (Hq + Hkv) if low < Hkv else 0) + stored(n, low)
            flops += 2.0 * d * Hq * (n + 1) * (n + 2)
            total += row * 2 * Hkv * (n + 1)
        return {"bytes": total, "flops": flops}
    dist, keep = n - P, case["keep"]
    for low in starts:
        total += fill(n, low)
        if low:
            total += row * low * n + 4 * low * dist * 2 + 4 * low * keep
            flops += 2.0 * d * case["obs"] * (Hq // Hkv) * low * n
        total += 2 * row * keep * (Hkv + low) + 2 * row * Hkv * (P + keep)
        flops += 4.0 * d * Hq * (P + keep)
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] == "similarity":
        return {"rel": 1e-5}      # 32-bit sums and logarithms; the values lie near 1
    # bf16 probabilities and outputs, 32-bit sums: another order of the sums moves an output by a bf16 step here and there
    return {"rel": 1e-2, "max": 6e-2}


# ---- the same in 64 bits ----

def _attend(case, q_own, q_low, k_own, k_low, v, pos, tau=None):
    """[rows][rep][d] of one kv head's query heads in 64 bits: q_* [rows][rep][d], k_*, v [n][d], pos [rows] (each query's position)."""
    rows, rep, d = q_own.shape
    n = v.shape[0]
    j = torch.arange(n, device=DEV)[None, :]
    i = pos[:, None]
    near = ((j < case["sink"]) | (j > i - case["window"])) & (j <= i)
    far = (j <= i) & ~near
    c = 1.0 / math.sqrt(d)
    out = torch.empty((rows, rep, d), dtype=torch.float64, device=DEV)
    for g in range(rep):
        a = (q_own[:, g].double() @ k_own.double().T) * c
        if bool(far.any()) and k_low is not None:
            a = torch.where(far, (q_low[:, g].double() @ k_low.double().T) * c, a)
        a = a.masked_fill(~(near | far), -math.inf)
        if tau is not None and k_low is not None:
            p, f = torch.logsumexp(a.masked_fill(~near, -math.inf), 1), torch.logsumexp(a.masked_fill(~far, -math.inf), 1)
            skip = 1.0 / (1.0 + torch.exp(f - p)) >= tau
            a = a.masked_fill(far & skip[:, None], -math.inf)
        out[:, g] = torch.softmax(a, dim=1) @ v.double()
    return out


def _by_head(t, case):
    return t.unflatten(1, (case["kv_heads"], -1))


def exact(case, seed):
    s = prepare({**case, "graph": False} if "graph" in case else case, seed)
    kind = case["kind"]
    if kind == "similarity":
        return _exact_similarity(s["att"])
    L, Hkv, d = case["layers"], case["kv_heads"], case["head_dim"]
    table = _table(case)
    if kind in ("prefill", "chunked"):
        outs, first = [], []
        for l in range(L):
            new = []
            out = torch.empty((case["n"], Hkv, case["q_heads"] // Hkv, d), dtype=torch.float64, device=DEV)
            for h in range(Hkv):
                low = table[l][h]
                q, ql = (_by_head(s["q"][x], case)[:, h] for x in (l, low))
                for a in range(0, case["n"], 2048):
                    z = slice(a, min(case["n"], a + 2048))
                    out[z, h] = _attend(case, q[z], ql[z], s["k"][l][:z.stop, h], s["k"][low][:z.stop, h] if low != l else None,
                                        s["v"][l][:z.stop, h], torch.arange(z.start, z.stop, device=DEV))
                q, ql = (_by_head(s["last"][x], case)[:, h] for x in (l, low))
                k, kl, v = (torch.cat([whole[:, h], one[:, h]]) for whole, one in
                            ((s["k"][l], s["k_new"][l]), (s["k"][low], s["k_new"][low]), (s["v"][l], s["v_new"][l])))
                new.append(_attend(case, q, ql, k, kl if low != l else None, v, torch.tensor([case["n"]], device=DEV)))
            outs.append(out.flatten(1, 2))
            first.append(torch.stack(new, 1).flatten(1, 2))
        return {"out": outs, "first": first}
    if kind == "selection":
        return {"votes": [_exact_votes(case, s, l) if l in table[l] else None for l in range(L)], "sel": None, "out": [None] * L}
    lens = _lens(case)
    T = case.get("tokens", 1)
    out = torch.empty((T, L, case["batch"], case["q_heads"], d), dtype=torch.float64, device=DEV)
    for l in range(L):
        for b, n in enumerate(lens):
            if kind == "steps":
                pos = torch.arange(n, n + T, device=DEV)
                q = [_by_head(torch.stack([s["q"][t][x][b] for t in range(T)]), case) for x in range(L)]
                k = [torch.cat([s["k"][x][b]] + [s["k_new"][t][x][b:b + 1] for t in range(T)]) for x in range(L)]
                v = torch.cat([s["v"][l][b]] + [s["v_new"][t][l][b:b + 1] for t in range(T)])
            else:
                pos = torch.tensor([n - 1], device=DEV)
                q = [_by_head(s["q"][x][b:b + 1], case) for x in range(L)]
                k, v = [s["k"][x][b] for x in range(L)], s["v"][l][b]
            heads = []
            for h in range(Hkv):
                low = table[l][h]
                heads.append(_attend(case, q[l][:, h], q[low][:, h], k[l][:, h], k[low][:, h] if low != l else None, v[:, h], pos,
                                     case.get("tau")))
            out[:, l, b] = torch.stack(heads, 1).flatten(1, 2)
    return out if kind == "steps" else {"out": [out[0, l] for l in range(L)], "skipped": None}


def _exact_votes(case, s, l):
    n, Hkv, obs = case["n"], case["kv_heads"], case["obs"]
    q = _by_head(s["q"][l], case)
    votes = torch.zeros((Hkv, n - case["sink"] - case["window"]), dtype=torch.float64, device=DEV)
    late = torch.arange(n, device=DEV)[None, :] > torch.arange(n - obs, n, device=DEV)[:, None]
    for h in range(Hkv):
        if _lowest(case, l, h) != l:
            continue
        for g in range(q.shape[2]):
            a = (q[:, h, g].double() @ s["k"][l][:, h].double().T) / math.sqrt(case["head_dim"])
            w = torch.softmax(a.masked_fill(late, -math.inf), dim=1).sum(0)
            votes[h] += w[case["sink"]:n - case["window"]]
    return votes


def _exact_similarity(att):
    L, H, R, _ = att.shape
    sim = torch.ones((H, L, L), dtype=torch.float64, device=DEV)
    for h in range(H):
        x = att[:, h].double()
        xlogx = torch.special.xlogy(x, x)
        for a in range(L - 1):
            later = slice(a + 1, L)
            m = 0.5 * (x[a:a + 1] + x[later])
            js = 0.5 * (xlogx[a:a + 1] + xlogx[later]) - torch.special.xlogy(m, m)
            v = 1.0 - js.sum(dim=(1, 2)) / (R * math.log(2.0))
            sim[h, a, later] = v
            sim[h, later, a] = v
    return sim
