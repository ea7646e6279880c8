"""The work that a program built on this library has it do, as cases that can be timed and compared.

A case is one pass through the public entry points (`Verifier`, `Drafter`, `ded_build_tree`) on inputs that are made
from a seed alone.  Four kinds:

  step       one verification step: `verify_step`, then `sample` where the case samples, then `accept`; a plain decoding
             step is a tree of one node, a chunk of a prompt is a chain whose nodes are all kept
  draft      the whole round of the decoding loop: tree search of the draft maker, pseudo-sequence, step, approval
  attention  the tree-attention entry point alone, called once for each layer, as a program with its own projections does
  cache      a stored prompt's K/V put into the cache and read back, layer by layer (prefix reuse)

The weights are random, N(0, 0.02) matrices with the residual projections scaled by 1 / sqrt(2 layers), unit-variance
embeddings and gains of 1 + N(0, 0.1); the LM head also holds a successor for every token, so that the model is as sure
of its next token as a trained one is (its logit stands about 15 above the others).  The drafts carry the successors
with probability 0.6 per node, so a step approves two to three tokens, the lengths that draft verification reaches in
use.  Prefix K/V are N(0, 1.28), the spread of the projections of a normalised input of width 4096.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2407_12021_amd import Verifier
from paper_2407_12021_amd.binding import Drafter, DED_OK, ded_build_tree


class _Model:
    """The model description that `Verifier` reads."""

    def __init__(self, case):
        self.name = "perf"
        self.n_layers, self.d_model = case["layers"], case["d"]
        self.n_heads, self.n_kv_heads, self.head_dim = case["heads"], case["kv_heads"], case["head_dim"]
        self.d_ffn, self.vocab = case["ffn"], case["vocab"]
        self.rope_base, self.rms_eps = case["rope_base"], 1e-5
        self.dtype = case["dtype"]


def _shape(dtype, layers, d, heads, kv_heads, head_dim, ffn, vocab, rope_base=10000.0):
    return {"dtype": dtype, "layers": layers, "d": d, "heads": heads, "kv_heads": kv_heads, "head_dim": head_dim,
            "ffn": ffn, "vocab": vocab, "rope_base": rope_base}


# the shapes of this repository's configurations, at their own depth
_TINY = _shape("fp32", 2, 256, 4, 4, 64, 688, 4096)
_SMALL = _shape("fp32", 4, 1024, 8, 8, 128, 2816, 8192)
_LLAMA2_7B = _shape("bf16", 32, 4096, 32, 32, 128, 11008, 32000)
_LLAMA2_13B = _shape("bf16", 40, 5120, 40, 40, 128, 13824, 32000)
_LLAMA3_8B = _shape("bf16", 32, 4096, 32, 8, 128, 14336, 128256, 500000.0)


def _step(shape, prefix, nodes, accept=0, logits=True, sample=False):
    """prefix / nodes: one number per sequence of the batch, as text ("1024" or "5000,777")."""
    return dict(shape, kind="step", prefix=prefix, nodes=nodes, accept=accept, logits=logits, sample=sample)


def _attention(layers, heads, kv_heads, prefix, nodes, static=False):
    return dict(_shape("bf16", layers, 128, heads, kv_heads, 128, 128, 16), kind="attention", prefix=prefix, nodes=nodes,
                static=static)


def _cache(layers, kv_heads, first, slots):
    return dict(_shape("bf16", layers, 128, kv_heads, kv_heads, 128, 128, 16), kind="cache", first=first, slots=slots)


def listed():
    def named(name, case):
        return dict(case, name=name)

    return [
        # the smallest call: a draft-sized fp32 model, where launches and the host path are all there is
        named("tiny_fp32", _step(_TINY, "128", "16")),
        # full precision at an ordinary size, a ragged batch of trees
        named("small_fp32", _step(_SMALL, "512,131,300,17", "48,21,64,7")),
        # plain decoding through the library: one node, one token (what every user does where the draft finds nothing)
        named("decode_7b", _step(_LLAMA2_7B, "1024", "1")),
        # the serving loop's step: 64-node tree on a 1024-token prefix, tokens only
        named("tree_7b", _step(_LLAMA2_7B, "1024", "64", logits=False)),
        # the whole round of the decoding loop with the draft maker, tree cut at 40 nodes
        named("drafted_7b", dict(_LLAMA2_7B, kind="draft", prefix="700", nodes="40")),
        # the pseudo-sequence of 24 candidates of 4 tokens that share nothing: 97 rows
        named("paper_7b", _step(_LLAMA2_7B, "1023", "97")),
        # a chunk of a prompt with the scores of its tokens
        named("prefill_7b", _step(_LLAMA2_7B, "768", "256", accept=1)),
        # a ragged batch with sampling on grouped-query heads and a large vocabulary
        named("sampled_8b", _step(_LLAMA3_8B, "5001,777,2900", "37,21,50", sample=True)),
        # batched trees of several sequences
        named("batch_13b", _step(_LLAMA2_13B, "2048,2048,2048,2048", "128,128,128,128")),
        # the largest: eight long contexts with large trees, tokens only
        named("batch_8b", _step(_LLAMA3_8B, ",".join(["16384"] * 8), ",".join(["256"] * 8), logits=False)),
        # attention alone, eight layers of a long context
        named("attention_7b", _attention(8, 32, 32, "4096", "64")),
        # a prompt's K/V restored into a cache and read out again, all layers
        named("cache_8b", _cache(32, 8, 0, 2001)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: sizes log-uniform, odd ones among them, never more work than the largest."""
    kind = rng.choice(["step", "step", "step", "batch", "batch", "fp32", "draft", "attention", "cache"])
    if kind == "fp32":
        head_dim = rng.choice([32, 64, 128])
        kv_heads = rng.choice([1, 2, 4, 8])
        heads = kv_heads * rng.choice([1, 2, 4])
        shape = _shape("fp32", rng.randint(1, 6), 64 * _log_int(rng, 2, 20), heads, kv_heads, head_dim,
                       16 * _log_int(rng, 12, 200), 16 * _log_int(rng, 20, 1000))
        batch = rng.randint(1, 4)
        return _step(shape, ",".join(str(_log_int(rng, 8, 1000)) for _ in range(batch)),
                     ",".join(str(_log_int(rng, 1, 100)) for _ in range(batch)), accept=0, logits=True)
    if kind == "attention":
        kv_heads = rng.choice([4, 8, 32, 40])
        heads = kv_heads if kv_heads >= 32 else kv_heads * 4
        batch = rng.choice([1, 1, 2, 3, 6])
        # the entry point with the library's own scratch takes calls whose buffers fit its 32 MiB: one ordinary tree
        static = batch == 1 and kv_heads >= 32 and rng.random() < 0.4
        return _attention(rng.randint(2, 8), heads, kv_heads, ",".join(str(_log_int(rng, 64, 12000)) for _ in range(batch)),
                          ",".join(str(_log_int(rng, 1, 64 if static else 200)) for _ in range(batch)), static=static)
    if kind == "cache":
        return _cache(rng.randint(2, 32), rng.choice([8, 32]), _log_int(rng, 1, 500) - 1, _log_int(rng, 1, 3000))
    shape = rng.choice([_LLAMA2_7B, _LLAMA3_8B, _LLAMA2_13B])
    if kind == "draft":
        return dict(shape, kind="draft", prefix=str(_log_int(rng, 64, 8000)), nodes=str(rng.randint(8, 40)))
    if kind == "step":
        return _step(shape, str(_log_int(rng, 16, 16000)), str(_log_int(rng, 1, 256)), accept=int(rng.random() < 0.2),
                     logits=rng.random() < 0.5, sample=rng.random() < 0.25)
    batch = rng.randint(2, 8)
    # without grouped-query heads a long batch's cache would not fit the card three times
    top = _log_int(rng, 128, 12000 if shape["kv_heads"] == 8 else 24000 // batch)
    most = _log_int(rng, 8, 200)
    return _step(shape, ",".join(str(max(1, int(top * rng.uniform(0.3, 1.0)))) for _ in range(batch)),
                 ",".join(str(max(1, int(most * rng.uniform(0.3, 1.0)))) for _ in range(batch)),
                 logits=rng.random() < 0.3, sample=rng.random() < 0.2)


def _ints(text):
    return [int(x) for x in str(text).split(",")]


def _weights(case, g, successor):
    """Random weights on the GPU in the case's storage type; the LM head's row of successor[t] leans on t's embedding."""
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    L, d, V, F = case["layers"], case["d"], case["vocab"], case["ffn"]
    q, kv = case["heads"] * case["head_dim"], case["kv_heads"] * case["head_dim"]

    def mat(rows, cols, std):
        return torch.empty(rows, cols, dtype=dt, device="cuda").normal_(0.0, std, generator=g)

    def gain():
        return 1.0 + 0.1 * torch.randn(d, device="cuda", generator=g)

    res = 0.02 / math.sqrt(2.0 * max(L, 1))
    layers = [{"wq": mat(q, d, 0.02), "wk": mat(kv, d, 0.02), "wv": mat(kv, d, 0.02), "wo": mat(d, q, res),
               "wg": mat(F, d, 0.02), "wu": mat(F, d, 0.02), "wd": mat(d, F, res), "norm_attn": gain(),
               "norm_ffn": gain()} for _ in range(L)]
    emb = mat(V, d, 1.0)
    head = mat(V, d, 0.02)
    at = torch.from_numpy(successor).cuda()
    head[at] += (30.0 / d) * emb
    return {"emb": emb, "lm_head": head, "final_norm": gain(), "layers": layers}


def _random_tree(r, n, chain):
    """parent[i] drawn from the nodes before i; a chain where every node is kept."""
    parent = np.arange(-1, n - 1, dtype=np.int32)
    if not chain:
        for i in range(1, n):
            parent[i] = int(r.integers(0, i))
    return parent


def _draft_tokens(r, parent, successor):
    """A child carries the successor of its parent's token with probability 0.6, unless an elder sibling has it."""
    token = r.integers(0, len(successor), size=len(parent)).astype(np.int32)
    taken = set()
    for i in range(1, len(parent)):
        p = int(parent[i])
        if p not in taken and r.random() < 0.6:
            token[i] = successor[token[p]]
            taken.add(p)
    return token


def _fill_cache(ver, case, prefix, g):
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    for b, p in enumerate(prefix):
        for layer in range(case["layers"] if p else 0):
            kv = torch.empty(2, case["kv_heads"], p, case["head_dim"], dtype=dt, device="cuda").normal_(0.0, 1.28, generator=g)
            ver.kv_store(layer, b, 0, kv[0], kv[1])


def _draft_corpus(drafter, r, vocab, successor, prev, root):
    """Tri-grams around the context (prev, root): four levels of six successors each, the model's own among them."""
    level = [(prev, root)]
    for _ in range(4):
        after = []
        for a, b in level:
            words = dict.fromkeys([int(successor[b])] + [int(x) for x in r.integers(0, vocab, size=5)])
            for w, times in zip(words, [60, 45, 35, 25, 18, 14]):
                drafter.count([a, b, w], times)
                after.append((b, w))
        level = after
    drafter.finalize(12)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = np.random.default_rng(seed)
    kind = case["kind"]
    model = _Model(case)
    successor = r.permutation(case["vocab"]).astype(np.int64)
    state = {"case": case}
    if kind == "cache":
        state["ver"] = Verifier(model, _weights(case, g, successor), max_batch=2, kv_capacity=case["first"] + case["slots"] + 64,
                                max_nodes=64)
        shape = (case["kv_heads"], case["slots"], 128)
        state["kv"] = [[torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.28, generator=g) for _ in range(2)]
                       for _ in range(case["layers"])]
        return state
    prefix, nodes = _ints(case["prefix"]), _ints(case["nodes"])
    most = max(nodes)
    ver = Verifier(model, _weights(case, g, successor), max_batch=len(prefix), kv_capacity=max(prefix) + most + 64, max_nodes=most)
    _fill_cache(ver, case, prefix, g)
    state.update(ver=ver, prefix=prefix)
    chain = bool(case.get("accept", 0))
    state["parents"] = [_random_tree(r, n, chain) for n in nodes]
    if kind == "attention":
        B = len(prefix)
        shape_q = (B, most, case["heads"], 128)
        shape_kv = (B, case["kv_heads"], most, 128)

        def unit(shape):
            return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0, generator=g)

        state["inputs"] = [(unit(shape_q), unit(shape_kv), unit(shape_kv)) for _ in range(case["layers"])]
        state["outs"] = [torch.zeros(shape_q, dtype=torch.bfloat16, device="cuda") for _ in range(case["layers"])]
        return state
    state["tokens"] = [_draft_tokens(r, p, successor) for p in state["parents"]]
    if kind == "draft":
        state["prev"], state["root"] = (int(x) for x in r.choice(case["vocab"], size=2, replace=False))
        state["uniform"] = r.random(600)
        state["drafter"] = Drafter()
        _draft_corpus(state["drafter"], r, case["vocab"], successor, state["prev"], state["root"])
    if case.get("sample"):
        state["uniform"] = [r.random(n).astype(np.float32) for n in nodes]
    return state


def _padded(rows, width):
    """The lists of `accept` as one array, so that every pass has the same outputs (-1 where a list has ended)."""
    out = np.full((len(rows), width), -1, np.int32)
    for b, row in enumerate(rows):
        out[b, : len(row)] = row
    return out


def run(state):
    case, ver = state["case"], state["ver"]
    kind = case["kind"]
    if kind == "cache":
        out = []
        for layer, (k, v) in enumerate(state["kv"]):
            ver.kv_store(layer, 1, case["first"], k, v)
        for layer in range(case["layers"]):
            out.append(ver.kv_load(layer, 1, case["first"], case["slots"]))
        return out
    if kind == "attention":
        return [ver.tree_attention(layer, state["prefix"], state["parents"], q, k, v, out=o, static=case["static"])
                for layer, ((q, k, v), o) in enumerate(zip(state["inputs"], state["outs"]))]
    width = ver.max_nodes + 1
    if kind == "draft":
        cands = [words for _, words in state["drafter"].mcts(state["prev"], state["root"], state["uniform"], iterations=150, l=4,
                                                             n=24, c1=32.0, c2=8.0)]
        rc, parent, token, _ = ded_build_tree(state["root"], cands, ver.max_nodes)
        assert rc == DED_OK
        logits = ver.verify_step(state["prefix"], [parent], [token], want_logits=True)
        tokens, path, length = ver.accept(mode=0)
        return {"logits": logits, "tree": _padded([parent, token], ver.max_nodes), "tokens": _padded(tokens, width),
                "path": _padded(path, width), "length": np.asarray(length, np.int32)}
    logits = ver.verify_step(state["prefix"], state["parents"], state["tokens"], want_logits=case["logits"])
    if case["sample"]:
        ver.sample(0.8, 0.9, state["uniform"])
    out = {}
    if logits is not None:
        out["logits"] = logits
    else:  # a loop that asks for no logits reads every node's token and how sure the model is of it
        out["argmax"], out["margin"] = ver.get_argmax()
    tokens, path, length = ver.accept(mode=case["accept"])
    out.update(tokens=_padded(tokens, width), path=_padded(path, width), length=np.asarray(length, np.int32))
    return out


def work(case):
    kind, hd, L = case["kind"], case["head_dim"], case["layers"]
    e = 2 if case["dtype"] == "bf16" else 4
    heads, kv_heads = case["heads"], case["kv_heads"]
    if kind == "cache":  # stored: read plain, write the cache; loaded: the other way round
        return {"bytes": 2 * 2 * L * 2 * kv_heads * case["slots"] * hd * e, "flops": 0}
    prefix, nodes = _ints(case["prefix"]), _ints(case["nodes"])
    rows = sum(nodes)
    seen = sum(n * p + n * (n + 1) // 2 for n, p in zip(nodes, prefix))  # keys inside the prefix, and ancestors at most
    attn_flops = 4 * L * heads * hd * seen
    attn_bytes = 2 * L * kv_heads * hd * e * sum(prefix)
    if kind == "attention":
        qo = 2 * L * rows * heads * hd * e
        return {"bytes": attn_bytes + qo + 2 * L * rows * kv_heads * hd * e, "flops": attn_flops}
    d, F, V = case["d"], case["ffn"], case["vocab"]
    per_layer = (2 * heads + 2 * kv_heads) * hd * d + 3 * d * F
    mats = L * per_layer + V * d
    written = 2 * L * rows * kv_heads * hd * e
    bytes_ = mats * e + rows * d * e + attn_bytes + written + (rows * V * 4 if kind == "draft" or case["logits"] else 0)
    return {"bytes": bytes_, "flops": 2 * rows * mats + attn_flops}


def tolerance(case):
    """About four times what the library was measured to be off from the same model in float64: 1.4e-7 (rel) and 7e-7 (max)
    in fp32; 3.2e-4 to 3.8e-4 and 2.0e-3 in the 16-bit path; 1.7e-3 and 4.3e-3 for attention, whose output is bf16."""
    if case["kind"] == "cache":
        return "exact"  # bf16 values come back as they were stored
    if case["dtype"] == "fp32":
        return {"rel": 1e-6, "max": 5e-6}
    if case["kind"] == "attention":
        return {"rel": 7e-3, "max": 2e-2}
    return {"rel": 1.5e-3, "max": 8e-3}
