"""Kernels at the sizes where their tiling, remainders and dispatch rules change, against the fp64 oracle."""
import numpy as np
import pytest

import ded_inputs as di
import oracle

pytestmark = pytest.mark.gpu


def _verifier(*a, **k):
    from paper_2407_12021_amd import Verifier
    return Verifier(*a, **k)


def _step_error(cfg, w, prefix_len, nodes, seed):
    """Largest logit error of one ragged batch step whose prefixes were computed by the library and the oracle each."""
    B, most = len(nodes), max(nodes)
    ver = _verifier(cfg, w, max_batch=B, kv_capacity=max(prefix_len) + most + 64, max_nodes=most)
    prefixes = [di.zipf_tokens(cfg.vocab, max(p, 1), seed=seed, stream=b)[:p] for b, p in enumerate(prefix_len)]
    caches = [oracle.prefill(cfg, w, t)[1:] if len(t) else None for t in prefixes]
    for b, c in enumerate(caches):
        for l in range(cfg.n_layers if c else 0):
            k, v = (np.ascontiguousarray(np.asarray(x[l], np.float32).transpose(1, 0, 2)) for x in c)
            if cfg.dtype == "bf16":
                k, v = di.f32_to_bf16_bits(k), di.f32_to_bf16_bits(v)
            ver.kv_store(l, b, 0, k, v)
    parents = [di.random_tree(n, None, seed=seed + b) for b, n in enumerate(nodes)]
    tokens = [di.zipf_tokens(cfg.vocab, n, seed=seed + 1, stream=b) for b, n in enumerate(nodes)]
    logits = ver.verify_step(prefix_len, parents, tokens, want_logits=True).cpu().numpy().astype(np.float64)
    ver.accept(mode=0)
    ver.close()
    worst = 0.0
    for b, n in enumerate(nodes):
        if caches[b]:
            pk, pv = ([oracle.widen(x) for x in c] for c in caches[b])
            if cfg.dtype == "bf16":
                pk, pv = ([di.round_to_bf16(np.asarray(x, np.float32)) for x in c] for c in (pk, pv))
        else:
            pk = pv = [np.zeros((0, cfg.n_kv_heads, cfg.head_dim))] * cfg.n_layers
        ref, _, _ = oracle.verify_tree(cfg, w, parents[b], tokens[b], pk, pv)
        worst = max(worst, float(np.abs(logits[b, :n] - ref).max()))
        assert not logits[b, n:].any()
    return worst


# (d, H, Hkv, hd, F, V), prefix lengths, tree sizes: k not a multiple of 4 (scalar loads) or of 32, features not a
# multiple of the tile, head dims on both sides of the fused rotary projection (32) and of the matrix-core attention (16),
# one and several row tiles, more feature tiles than one per CU
FP32_EDGES = [
    ((33, 2, 2, 8, 17, 50), [0, 5], [1, 16]),
    ((36, 2, 1, 16, 50, 101), [33], [17]),
    ((64, 4, 1, 32, 44, 500), [15, 17, 0], [16, 3, 33]),
    ((132, 2, 2, 64, 340, 97), [127, 64, 1, 130], [1, 16, 17, 48]),
    ((256, 3, 1, 128, 688, 4096), [129], [16]),
    ((320, 2, 1, 256, 96, 6000), [31, 300], [65, 130]),
]


@pytest.mark.parametrize("case", range(len(FP32_EDGES)))
def test_fp32_projections_and_attention_at_tile_edges(case):
    """Bound: the fp32 path's 1e-4 logit tolerance (sums of at most 688 products of O(1) terms round to ~1e-6)."""
    (d, H, Hkv, hd, F, V), prefix_len, nodes = FP32_EDGES[case]
    cfg = di.ModelConfig(f"f32-edge{case}", 2, d, H, Hkv, hd, F, V, dtype="fp32")
    w = di.make_weights(cfg, seed=40 + case, gain_jitter=0.1, std=0.05)
    err = _step_error(cfg, w, prefix_len, nodes, seed=50 + case)
    print(f"max |logit error| {err:.2e}")
    assert err <= 1e-4
