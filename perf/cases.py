"""Workloads of the draft-tree step, for timing it and for comparing two builds' results.

A case is one decoding round as a serving loop runs it: log-probabilities and top tokens of the
drafter's rows, the draft tree, attention of every tree node over the cache and its ancestors (once
per target layer), the walk over the target's logits and, where the loop keeps its cache in place,
the append of the accepted rows.  Fields of a case:

  batch, B, V, N     sequences, draft positions, vocabulary, node budget
  Hq, Hkv, D, dtype  query heads, KV heads, head size, "bf16" or "fp32"
  L_lo, L_hi         cached rows of a sequence, uniform between the two
  layers             attention calls of the round, each with its own cache
  p                  probability of each draft row's top token; 0: the nearly flat rows of bench.py
  temperature        of the target's decoding; 0: greedy
  append             the cache has room behind each sequence and takes the accepted rows in place
  deferred           the calls are marshalled once and kept, as a tight loop does; otherwise each
                     call marshals its arguments and allocates its results
"""
import heapq
import math

import numpy as np
import torch

import ddtree_inputs as di
import paper_2604_12989_amd as dd

_BF16_128 = dict(B=16, V=151936, Hq=32, Hkv=8, D=128, dtype="bf16")


def _case(name, **kw):
    c = dict(name=name, batch=1, layers=1, p=0.0, temperature=0.0, append=False, deferred=True)
    c.update(kw)
    return c


def _config(name, number, **kw):
    """One of the shapes in ddtree_inputs.CONFIGS."""
    c = dict(di.CONFIGS[number])
    lo, hi = c["L"] if isinstance(c["L"], tuple) else (c["L"], c["L"])
    del c["name"], c["L"]
    return _case(name, L_lo=lo, L_hi=hi, **{**c, **kw})


def listed():
    return [
        # A model of a few million weights in fp32: every kernel at its latency.
        _config("tiny_fp32", 1),
        # The smallest budget of the sweep right behind a short prompt.
        _case("budget16_short", **_BF16_128, N=16, L_lo=300, L_hi=300, p=0.8, append=True),
        # The four shapes that bench.py knows: chat turn, the headline, long document, a batch.
        _config("n64_l2k", 2),
        _config("n256_l8k", 3),
        _config("n512_l32k", 4),
        _config("batch16_ragged", 5),
        # The headline shape with a confident drafter, in a loop that keeps its cache in place.
        _config("n256_l8k_confident", 3, p=0.9, append=True),
        # The largest budget that the library takes.
        _case("n1024_l8k", **_BF16_128, N=1024, L_lo=8192, L_hi=8192, p=0.7, append=True),
        # A round over several target layers, odd sizes, as a model's forward calls the library:
        # attention is called per layer, the rest once a round.
        _case("layers8_odd", B=16, V=151936, N=60, Hq=32, Hkv=8, D=128, dtype="bf16", L_lo=3001,
              L_hi=3001, layers=8, p=0.8, append=True, deferred=False),
        # A few ragged sequences, a vocabulary that no vector width divides, a short block.
        _case("batch4_odd", batch=4, B=7, V=50021, N=100, Hq=24, Hkv=8, D=128, dtype="bf16",
              L_lo=37, L_hi=3001, p=0.6, append=True, deferred=False),
        # A target that samples.
        _case("sampled_batch2", batch=2, **_BF16_128, N=128, L_lo=1000, L_hi=4096, p=0.7,
              temperature=0.8, append=True),
        # Heads of 64.
        _case("head64_n64_l2k", B=16, V=32003, N=64, Hq=16, Hkv=4, D=64, dtype="bf16", L_lo=2047,
              L_hi=2047, layers=2, p=0.7, append=True),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _cost(c):
    """Rough time of a pass, in units of one byte moved: the heads that the matrix cores serve at a
    rate of their own, all others (fp32, other head sizes) at a vector unit's."""
    w = work(c)
    return w["bytes"] + w["flops"] / (200 if (c["dtype"], c["D"]) == ("bf16", 128) else 2)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choices(["bf16", "head64", "fp32"], [8, 2, 1])[0]
        Hkv = rng.choice([1, 2, 4, 8]) if kind != "bf16" else rng.choice([4, 8, 8])
        group = rng.choice([1, 2, 3, 4, 4, 4, 5, 7, 8])
        hi = 32768 if kind == "bf16" else 4096 if kind == "head64" else 512
        a, b = _log_int(rng, 32, hi), _log_int(rng, 32, hi)
        c = _case("", batch=rng.choice([1, 1, 1, 2, 3, 4, 7, 16]), B=rng.randint(4, 24),
                  V=_log_int(rng, 1000, 160000) if rng.random() < 0.6 else 151936,
                  N=_log_int(rng, 8, 1024 if kind == "bf16" else 256), Hq=Hkv * group, Hkv=Hkv,
                  D=128 if kind == "bf16" else 64, dtype="fp32" if kind == "fp32" else "bf16",
                  L_lo=min(a, b), L_hi=max(a, b), layers=rng.choice([1, 1, 2, 4]),
                  p=rng.choice([0.0, round(rng.uniform(0.3, 0.95), 2), round(rng.uniform(0.3, 0.95), 2)]),
                  temperature=rng.choice([0.0, 0.0, 0.0, round(rng.uniform(0.3, 1.5), 2)]),
                  append=rng.random() < 0.6, deferred=rng.random() < 0.7)
        del c["name"]
        if _cost(c) <= most:
            return c


def _tree_depths(lp, N):
    """Depth of each node of the draft tree over the rows' sorted log-probabilities, in the order
    in which best-first search takes the nodes."""
    depth, heap, n = [0], [(-lp[0][0], 0, 0, 0.0)], 0
    while heap and len(depth) <= N:
        cost, d, r, above = heapq.heappop(heap)
        depth.append(d + 1)
        if r + 1 < len(lp[d]):
            heapq.heappush(heap, (-(above + lp[d][r + 1]), d, r + 1, above))
        if d + 1 < len(lp):
            heapq.heappush(heap, (-(-cost + lp[d + 1][0]), d + 1, 0, -cost))
    return depth


def _draft_logits(c, gen):
    """bench.py's rows (scale 3 * 0.85^d, one token raised by 4), or, with p > 0, that token raised
    until it holds probability p."""
    B, V = c["B"], c["V"]
    scale = 3.0 * 0.85 ** torch.arange(B, device="cuda", dtype=torch.float32)
    x = torch.randn((c["batch"], B, V), generator=gen, device="cuda") * scale[None, :, None]
    spike = torch.randint(V, (c["batch"], B, 1), generator=gen, device="cuda")
    if c["p"] > 0:
        others = x.scatter(2, spike, -math.inf).logsumexp(2, keepdim=True)
        return x.scatter(2, spike, others + math.log(c["p"] / (1 - c["p"])))
    return x.scatter_add(2, spike, torch.full_like(spike, 4.0, dtype=torch.float32))


def _target_logits(c, x, gen):
    """N(0,1) with 10 planted, in a share 0.8^depth of the rows, on the token that the drafter
    holds most likely at the next position."""
    batch, B, N, T = c["batch"], c["B"], c["N"], c["N"] + 1
    t = torch.randn((batch, T, c["V"]), generator=gen, device="cuda")
    top, tok = torch.log_softmax(x, 2).topk(min(N, c["V"]), dim=2)
    top, tok = top.cpu().tolist(), tok[:, :, 0].cpu().numpy()
    u = torch.rand((batch, T), generator=gen, device="cuda").cpu().numpy()
    rows, cols = [], []
    for s in range(batch):
        for i, d in enumerate(_tree_depths(top[s], N)):
            if d < B and u[s, i] < 0.8 ** d:
                rows.append(s * T + i)
                cols.append(tok[s, d])
    if rows:
        t.view(batch * T, -1)[torch.tensor(rows, device="cuda"), torch.tensor(np.array(cols), device="cuda")] = 10.0
    return t


class State:
    pass


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    batch, B, V, N, Hq, Hkv, D = (c[k] for k in ("batch", "B", "V", "N", "Hq", "Hkv", "D"))
    T, K = N + 1, min(N, V)
    tdt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32

    def randn(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(tdt)

    s = State()
    s.c = c
    lens = c["L_lo"] + di.randint(seed, 4000, batch, c["L_hi"] - c["L_lo"] + 1)
    # In place: a slot for the longest sequence and an accepted path each.  Otherwise packed.
    slot = c["L_hi"] + B + 1
    s.kv_offset = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    s.kv_start, s.kv_len = (slot * np.arange(batch)).astype(np.int32), lens.astype(np.int32)
    s.dst_row = (s.kv_start + s.kv_len).astype(np.int32)
    s.draft = _draft_logits(c, gen)
    s.target = _target_logits(c, s.draft, gen)
    s.root = torch.randint(V, (batch,), generator=gen, device="cuda").to(torch.int32)
    rows = slot * batch if c["append"] else int(s.kv_offset[-1])
    s.layers = [dict(q=randn(batch * T, Hq, D), k_cache=randn(rows, Hkv, D), v_cache=randn(rows, Hkv, D),
                     k_tree=randn(batch * T, Hkv, D), v_tree=randn(batch * T, Hkv, D))
                for _ in range(c["layers"])]
    s.ws = dd.Workspace(batch, B, V, N, Hq, Hkv, D, int(lens.sum()))
    s.calls = None
    if c["deferred"]:
        s.calls = _enqueue(s, defer=True)
    return s


def _attention(s, layer, mask, **kw):
    c = s.c
    dtype = dd.DTYPE_BF16 if c["dtype"] == "bf16" else dd.DTYPE_FP32
    where = (s.kv_start, s.kv_len) if c["append"] else (s.kv_offset,)
    f = dd.verify_attn_spans if c["append"] else dd.verify_attn
    return f(layer["q"], layer["k_cache"], layer["v_cache"], layer["k_tree"], layer["v_tree"], mask,
             *where, c["batch"], c["N"] + 1, c["Hq"], c["Hkv"], c["D"], 1.0 / math.sqrt(c["D"]), dtype,
             s.ws, **kw)


def _accept_options(c):
    return dict(temperature=c["temperature"], seed=12345) if c["temperature"] > 0 else {}


def _enqueue(s, defer=False):
    """The round's calls in order; deferred: the calls themselves and the buffers they fill."""
    c = s.c
    batch, B, N, T = c["batch"], c["B"], c["N"], c["N"] + 1
    K = min(N, c["V"])
    if not defer:
        tok, lp = dd.topk(s.draft, K, s.ws)
        tree = dd.build(tok, lp, N, s.root, s.ws)
        out = [_attention(s, layer, tree["ancestor_mask"]) for layer in s.layers]
        walk = dd.accept(s.target, tree["tokens"], tree["parent"], tree["depth"], tree["n_nodes"], B, s.ws,
                         **_accept_options(c))
        return tok, lp, tree, out, walk

    def ints(*shape):
        return torch.empty(shape, dtype=torch.int32, device="cuda")

    tok, lp = ints(batch, B, K), torch.empty((batch, B, K), device="cuda")
    tree = dict(tokens=ints(batch, T), parent=ints(batch, T), depth=ints(batch, T), rank=ints(batch, T),
                node_score=torch.empty((batch, T), device="cuda"),
                ancestor_mask=torch.empty((batch, T, (T + 63) // 64), dtype=torch.int64, device="cuda"),
                n_nodes=ints(batch))
    walk = dict(path=ints(batch, B + 1), n_accepted=ints(batch), bonus_token=ints(batch), posterior=ints(batch, T))
    out = [torch.empty_like(layer["q"]) for layer in s.layers]
    calls = [dd.topk(s.draft, K, s.ws, tok, lp, defer=True), dd.build(tok, lp, N, s.root, s.ws, out=tree, defer=True)]
    calls += [_attention(s, layer, tree["ancestor_mask"], out=o, defer=True) for layer, o in zip(s.layers, out)]
    calls.append(dd.accept(s.target, tree["tokens"], tree["parent"], tree["depth"], tree["n_nodes"], B, s.ws,
                           out=walk, defer=True, **_accept_options(c)))
    return calls, (tok, lp, tree, out, walk)


def run(s):
    c = s.c
    if s.calls is not None:
        calls, results = s.calls
        for call in calls:
            call()
    else:
        results = _enqueue(s)
    tok, lp, tree, out, walk = results
    r = dict(tok=tok, lp=lp, tree=tree, out=out, walk=walk)
    if c["append"]:
        for layer in s.layers:
            dd.compact(layer["k_tree"], layer["v_tree"], walk["path"], walk["n_accepted"], s.dst_row, c["batch"],
                       c["N"] + 1, c["B"], c["Hkv"], c["D"], layer["k_cache"], layer["v_cache"])
        r["cache"] = [(layer["k_cache"], layer["v_cache"]) for layer in s.layers]
    return r


def work(case):
    """Logits of both models, cache, tree rows and queries read once; results written once.  The
    attention's products over the mean cache length and, for the tree's part, a few ancestors a node."""
    c = case
    T, K = c["N"] + 1, min(c["N"], c["V"])
    e = 2 if c["dtype"] == "bf16" else 4
    L = (c["L_lo"] + c["L_hi"]) / 2
    once = 4 * c["V"] * (c["B"] + T) + 8 * c["B"] * K + T * (24 + 8 * ((T + 63) // 64))
    layer = e * c["D"] * (2 * L * c["Hkv"] + 2 * T * c["Hkv"] + 2 * T * c["Hq"])
    flops = 4 * c["D"] * c["Hq"] * T * (L + 3)
    return {"bytes": c["batch"] * (once + c["layers"] * layer), "flops": c["batch"] * c["layers"] * flops}


def tolerance(case):
    """Tokens, trees, masks and walks are defined exactly; a sampled token may go either way where two
    keys lie within the rounding of their fp32 arithmetic.  Attention in bf16: weights and results
    are rounded to bf16, partial results of split key ranges to fp16: 2.3e-3 (at most 0.03 of the
    root mean square) off the same attention in fp64, over all the bf16 cases.  In fp32 sums in
    another order: 5e-7 (8e-6) off."""
    t = {"rel": 1e-2, "max": 0.1} if case["dtype"] == "bf16" else {"rel": 2e-6, "max": 3e-5}
    if case["temperature"] > 0:
        t["differ"] = 0.004
    return t
