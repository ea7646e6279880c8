"""Kernels at the sizes where their tiling, remainders and dispatch rules change, against the fp64 oracle."""
import numpy as np
import pytest

import ded_inputs as di
import oracle

pytestmark = pytest.mark.gpu


def _verifier(*a, **k):
    from paper_2407_12021_amd import Verifier
    return Verifier(*a, **k)


def _check_argmax(logits, tokens, margins, nodes):
    """Tokens and margins of a step's real nodes are those of its fp32 logits, bit for bit: lowest id of the largest, largest minus
    second largest."""
    for b, n in enumerate(nodes):
        rows = logits[b, :n]
        top2 = np.partition(rows, -2, axis=1)[:, -2:]
        assert np.array_equal(tokens[b, :n], np.argmax(rows, axis=1)), b
        assert np.array_equal(margins[b, :n], top2[:, 1] - top2[:, 0]), b


def _step_error(cfg, w, prefix_len, nodes, seed):
    """Largest logit error of one ragged batch step whose prefixes were computed by the library and the oracle each; its tokens
    and margins have to be those of its logits."""
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
    logits = ver.verify_step(prefix_len, parents, tokens, want_logits=True).cpu().numpy()
    _check_argmax(logits, *ver.get_argmax(), nodes)
    logits = logits.astype(np.float64)
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
# one and several row tiles, more feature tiles than one per CU, 256 keys (the most in one range) and 257, more than 8 ranges of 128
FP32_EDGES = [
    ((33, 2, 2, 8, 17, 50), [0, 5], [1, 16]),
    ((36, 2, 1, 16, 50, 101), [33], [17]),
    ((64, 4, 1, 32, 44, 500), [15, 17, 0], [16, 3, 33]),
    ((132, 2, 2, 64, 340, 97), [127, 64, 1, 130], [1, 16, 17, 48]),
    ((256, 3, 1, 128, 688, 4096), [129], [16]),
    ((320, 2, 1, 256, 96, 6000), [31, 300], [65, 130]),
    ((64, 2, 1, 32, 44, 500), [240, 241, 1100], [16, 16, 20]),
    ((256, 2, 2, 128, 64, 97), [1010, 500, 245], [5, 33, 12]),
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


# the packed operands' larger tiles, with feature and row tiles that do not divide into them: 4 x 2 in gate/up and LM head over
# fewer k tiles than wavefronts (K = 52); 4 x 2, then 2 x 2, over an odd number of k tiles (K = 1040)
FP32_TILES = [
    ((52, 4, 2, 32, 2810, 16003), [7, 40, 3], [33, 61, 17]),
    ((1040, 2, 2, 64, 48, 8190), [5, 20], [16, 48]),
    ((1040, 2, 1, 64, 100, 4090), [9], [50]),
]


@pytest.mark.parametrize("case", range(len(FP32_TILES)))
def test_fp32_projections_of_every_tile(case):
    """Bound: sums of at most 2810 products of O(1) terms round to ~1e-5; the fp32 path's 1e-4 logit tolerance."""
    (d, H, Hkv, hd, F, V), prefix_len, nodes = FP32_TILES[case]
    cfg = di.ModelConfig(f"f32-tile{case}", 2, d, H, Hkv, hd, F, V, dtype="fp32")
    w = di.make_weights(cfg, seed=70 + case, gain_jitter=0.1, std=0.05)
    err = _step_error(cfg, w, prefix_len, nodes, seed=80 + case)
    print(f"max |logit error| {err:.2e}")
    assert err <= 1e-4


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_cache_rows_come_back_and_neighbours_stay(dtype):
    """Ranges that start, end or lie inside a 32-slot group of the cache: rows come back bit for bit (bf16 values widen to
    half and back exactly from 2^-14 up), and no slot beside the range changes."""
    import torch
    hd = 128 if dtype == "bf16" else 64
    cfg = di.ModelConfig("kv-edge-" + dtype, 1, 128, 4, 2, hd, 128, 64, dtype=dtype)
    cap = 192
    ver = _verifier(cfg, di.make_weights(cfg, seed=3), max_batch=2, kv_capacity=cap, max_nodes=16)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(5)

    def rows(n):
        x = torch.randn(2, n, hd, device="cuda", generator=g).to(dt)
        return torch.where(x.abs() < 2.0 ** -14, torch.ones_like(x), x)

    want = [rows(cap), rows(cap)]
    ver.kv_store(0, 1, 0, *want)
    for first, n in ((0, 1), (31, 1), (31, 2), (1, 31), (32, 32), (7, 100), (64, 96), (8, 8), (12, 8), (191, 1), (0, 192)):
        new = [rows(n), rows(n)]
        ver.kv_store(0, 1, first, new[0], new[1])
        for w, x in zip(want, new):
            w[:, first:first + n] = x
        for got, w in zip(ver.kv_load(0, 1, 0, cap), want):
            assert torch.equal(got, w), (first, n)
        for got, w in zip(ver.kv_load(0, 1, first, n), want):
            assert torch.equal(got, w[:, first:first + n]), (first, n)
    assert not any(x.any() for x in ver.kv_load(0, 0, 0, cap))  # the other sequence
    ver.close()


@pytest.mark.parametrize("V", [48, 1008, 4096 + 16, 36880, 262144 + 32])
def test_sampler_vocabularies(V):
    """Vocabularies below one pass of the workgroup, off its 4-id and 256-id granules, and above the 1024 sub-blocks of the
    inverse CDF, against the fp64 sampler on the same logits.  A decision counts where u is clear of every CDF step and of
    the nucleus boundary by 1e-5: the kernel's sums are exact to V 2^-40, its weights to some 1e-6 relative."""
    cfg = di.ModelConfig(f"samp-v{V}", 1, 128, 1, 1, 128, 128, V, dtype="bf16")
    w = di.make_weights(cfg, seed=8, std=0.3)
    ver = _verifier(cfg, w, max_batch=2, kv_capacity=64, max_nodes=24)
    nodes = [5, 24]
    parents = [di.random_tree(n, None, seed=n) for n in nodes]
    tokens = [di.zipf_tokens(V, n, seed=9, stream=b) for b, n in enumerate(nodes)]
    logits = ver.verify_step([0, 0], parents, tokens, want_logits=True).cpu().numpy().astype(np.float64)
    r = np.random.default_rng(1)
    decided = 0
    for temperature, top_p in ((1.0, 1.0), (0.4, 0.9), (0.7, 0.3), (2.5, 0.8)):
        us = [r.random(n).astype(np.float32) for n in nodes]
        ver.sample(temperature, top_p, us)
        got, _ = ver.get_argmax()
        for b, n in enumerate(nodes):
            ref, info = oracle.sample_rows(logits[b, :n], temperature, top_p, us[b].astype(np.float64))
            for i in range(n):
                edge = info[i]["edge_mass"] if info[i]["nucleus_slack"] <= 1e-5 else 0.0
                if info[i]["cdf_slack"] > 1e-5 + edge:
                    assert int(got[b, i]) == int(ref[i]), (temperature, top_p, b, i)
                    decided += 1
    assert decided >= 0.6 * 4 * sum(nodes), decided
    ver.accept(mode=0)
    ver.close()


# (d, H, Hkv, F, V), prefix lengths, tree sizes: k ranges shorter than the ring and not a multiple of it (K = 128, 384, 640),
# feature groups and rows that fill no whole tile (odd groups, 224 - 624 rows), tiles split over k 2 - 4 ways and whole,
# single-plane and two-plane LM heads (from 256 rows on)
TILE_EDGES = [
    ((128, 1, 1, 128, 80), [3, 0], [70, 130]),
    ((384, 3, 3, 640, 208), [17], [250]),
    ((256, 4, 1, 384, 1040), [9, 40, 0], [64, 65, 130]),
    ((640, 4, 2, 896, 5200), [5, 70], [200, 150]),
    ((1024, 8, 8, 2816, 8192), [20], [256]),
    ((512, 8, 2, 1408, 16400), [8, 3, 0], [250, 130, 220]),
]


@pytest.mark.parametrize("case", range(len(TILE_EDGES)))
def test_projections_at_tile_edges(case):
    """256 and more rows (trees padded to the largest).  Bound: the 16-bit path's 2e-2 logit tolerance (f16 rounding of weights' products and of the
    attention and SwiGLU outputs, 2^-12 each, on logits of a few units)."""
    (d, H, Hkv, F, V), prefix_len, nodes = TILE_EDGES[case]
    cfg = di.ModelConfig(f"tile-edge{case}", 2, d, H, Hkv, 128, F, V, dtype="bf16")
    w = di.make_weights(cfg, seed=60 + case, gain_jitter=0.1)
    err = _step_error(cfg, w, prefix_len, nodes, seed=70 + case)
    print(f"max |logit error| {err:.2e}")
    assert err <= 2e-2


# (d, H, Hkv, F, V) of one layer, prefix lengths, tree sizes, (tile, k ranges) of the down projection: residual projections whose slices
# are added by a launch of their own.  All three tiles, surplus row blocks, two row tiles, 64 packed rows that are summed like
# 128, 3 to 8 ranges that are and are not multiples of the ring
APART_EDGES = [
    ((1024, 8, 8, 2816, 1040), [5], [250], (4, 5)),
    ((2048, 16, 4, 8192, 1040), [3, 0], [70, 130], (4, 8)),
    ((1024, 8, 8, 1664, 1040), [0, 9], [256, 30], (5, 3)),
    ((4096, 32, 8, 14336, 1040), [7], [150], (5, 8)),
    ((4096, 32, 8, 14336, 1040), [7, 0], [48, 16], (6, 8)),
]


@pytest.mark.parametrize("case", range(len(APART_EDGES)))
def test_residual_projections_summed_apart(case):
    """Bound: the 16-bit path's 2e-2 logit tolerance, as above."""
    import ctypes as C

    from paper_2407_12021_amd import binding

    class Plan(C.Structure):
        _fields_ = [(n, C.c_int) for n in ("nwn", "nw", "splits", "tile", "whole", "ssq_waves")]

    (d, H, Hkv, F, V), prefix_len, nodes, (tile, ranges) = APART_EDGES[case]
    up = lambda x, to: -(-x // to) * to
    sum_rows, rows = up(len(nodes) * up(max(nodes), 16), 64), up(sum(up(n, 16) for n in nodes), 64)
    f = binding.lib()["_ZN3ded23bf16_gemm_plan_residualEiiiiil"]
    f.restype, f.argtypes = Plan, [C.c_int] * 5 + [C.c_int64]
    plan = f(sum_rows, rows, d, F, 8, 2 * F * max(512, sum_rows))
    assert (plan.tile, plan.splits, plan.whole) == (tile, ranges, -1)
    cfg = di.ModelConfig(f"apart-edge{case}", 1, d, H, Hkv, 128, F, V, dtype="bf16")
    w = di.make_weights(cfg, seed=200 + case, gain_jitter=0.1, threads=16)
    err = _step_error(cfg, w, prefix_len, nodes, seed=210 + case)
    print(f"max |logit error| {err:.2e}")
    assert err <= 2e-2


# (d, H, Hkv, F, V) of one layer, prefix lengths, tree sizes, (N, K) of the projections that the tile kernel runs: steps of 97,
# 144, 70 and 176 rows whose unsplit products run as two k ranges of the tile kernel, rows that fill no whole tile (wavefronts
# without rows, and with a surplus block), a vocabulary that ends inside a feature group
MID_EDGES = [
    ((2048, 16, 4, 8192, 65552), [5], [97], [(16384, 2048), (65552, 2048)]),
    ((4096, 32, 8, 14336, 32016), [3, 0, 40], [37, 21, 50], [(28672, 4096), (32016, 4096)]),
    ((5120, 40, 40, 1408, 1040), [9], [70], [(15360, 5120)]),
    ((4096, 32, 8, 14336, 32016), [7, 0, 9], [64, 50, 48], [(28672, 4096), (32016, 4096)]),
]


@pytest.mark.parametrize("case", range(len(MID_EDGES)))
def test_projections_of_65_to_255_rows(case, gemm_plan):
    """Bound: the 16-bit path's 2e-2 logit tolerance, as above; tokens and margins, with logits and without, are those of the logits."""
    (d, H, Hkv, F, V), prefix_len, nodes, tiled = MID_EDGES[case]
    rows = -(-len(nodes) * (-(-max(nodes) // 16) * 16) // 64) * 64
    for N, K in tiled:
        assert gemm_plan(rows, rows, N, K, 2, 4, N * 512).tile
    cfg = di.ModelConfig(f"mid-edge{case}", 1, d, H, Hkv, 128, F, V, dtype="bf16")
    w = di.make_weights(cfg, seed=100 + case, gain_jitter=0.1, threads=16)
    err = _step_error(cfg, w, prefix_len, nodes, seed=110 + case)
    print(f"max |logit error| {err:.2e}")
    assert err <= 2e-2
    ver = _verifier(cfg, w, max_batch=len(nodes), kv_capacity=128, max_nodes=max(nodes))
    parents = [di.random_tree(n, None, seed=b) for b, n in enumerate(nodes)]
    tokens = [di.zipf_tokens(V, n, seed=6, stream=b) for b, n in enumerate(nodes)]
    logits = ver.verify_step([0] * len(nodes), parents, tokens, want_logits=True).cpu().numpy()
    _check_argmax(logits, *ver.get_argmax(), nodes)
    ver.verify_step([0] * len(nodes), parents, tokens)
    _check_argmax(logits, *ver.get_argmax(), nodes)
    ver.close()


# (layers, d, H, Hkv, F, V), prefix lengths, tree sizes: steps of 16 and 32 padded rows; k ranges of one step of 128, ranges that
# are no multiple of the ring, half groups and whole groups (160 feature groups and more), 2 to 16 ranges per workgroup, a
# vocabulary that ends inside a group
SLIM_EDGES = [
    ((2, 128, 1, 1, 128, 80), [5], [1]),
    ((2, 384, 3, 1, 640, 208), [0, 33], [16, 9]),
    ((2, 640, 5, 5, 896, 1040), [70], [32]),
    ((1, 4096, 32, 32, 11008, 32048), [19], [1]),
    ((1, 4096, 32, 8, 14336, 32048), [40], [17]),
]


@pytest.mark.parametrize("case", range(len(SLIM_EDGES)))
def test_projections_of_few_rows(case):
    """Bound: the 16-bit path's 2e-2 logit tolerance, as above."""
    (L, d, H, Hkv, F, V), prefix_len, nodes = SLIM_EDGES[case]
    cfg = di.ModelConfig(f"slim-edge{case}", L, d, H, Hkv, 128, F, V, dtype="bf16")
    w = di.make_weights(cfg, seed=80 + case, gain_jitter=0.1, threads=16)
    err = _step_error(cfg, w, prefix_len, nodes, seed=90 + case)
    print(f"max |logit error| {err:.2e}")
    assert err <= 2e-2


# (d, H, Hkv, F, V), tree size: 3 - 11 row blocks in one to three groups of 2, 3 and 4; k ranges of four steps and more, of whole
# turns of the stream kernel's ring and half a turn more, in one slice and several; the last two in more workgroups than CUs too
# (down 768; gate/up 768 and down 480).  The wide kernel: WIDE_EDGES
GROUP_EDGES = [((128, 1, 1, 128, 80), 33)] + [((640, 5, 5, 896, 1040), n) for n in (48, 49, 65, 81, 97, 129, 145, 161)] + [
    ((4096, 32, 8, 11008, 4112), 40), ((4096, 32, 32, 11008, 4112), 145), ((2048, 16, 8, 8192, 1040), 145)]


@pytest.mark.parametrize("case", range(len(GROUP_EDGES)))
def test_projections_of_uneven_row_groups(case):
    """Bound: the 16-bit path's 2e-2 logit tolerance, as above."""
    (d, H, Hkv, F, V), n = GROUP_EDGES[case]
    cfg = di.ModelConfig(f"group-edge{case}", 1, d, H, Hkv, 128, F, V, dtype="bf16")
    w = di.make_weights(cfg, seed=120 + case, gain_jitter=0.1, threads=16)
    err = _step_error(cfg, w, [7], [n], seed=140 + case)
    print(f"max |logit error| {err:.2e}")
    assert err <= 2e-2


# (d, H, Hkv, F, V), tree size, {(N, K): (feature groups per workgroup, slices)} of the projections that the wide kernel runs: row
# blocks 3 (one group), 3 + 2, 4 + 3, 3 + 3 + 3, 4 + 3 + 3 and 4 + 4 + 3; two, three and four feature groups, the last ones surplus or
# ending inside a group; one slice and several, at most one workgroup per CU and more
WIDE_EDGES = [
    ((1024, 8, 8, 2816, 8208), 40, {(8208, 1024): (2, 3)}),
    ((1024, 8, 8, 2816, 8208), 65, {(8208, 1024): (2, 1)}),
    ((1024, 8, 8, 2816, 32016), 80, {(32016, 1024): (4, 1)}),
    ((1024, 8, 8, 2816, 32016), 97, {(32016, 1024): (4, 1)}),
    ((1024, 8, 8, 2816, 32016), 144, {(32016, 1024): (3, 1), (5632, 1024): (2, 1)}),
    ((1024, 8, 8, 2816, 32016), 160, {(32016, 1024): (3, 1), (5632, 1024): (2, 1)}),
    ((4096, 32, 32, 11008, 4112), 65, {(12288, 4096): (3, 2), (22016, 4096): (3, 1), (4112, 4096): (3, 5)}),
    ((4096, 32, 32, 11008, 4112), 176, {(22016, 4096): (3, 2)}),
    ((4096, 32, 8, 14336, 1040), 40, {(6144, 4096): (3, 8), (28672, 4096): (4, 2)}),
    ((4096, 32, 8, 14336, 1040), 97, {(6144, 4096): (3, 4), (28672, 4096): (4, 1)}),
    ((4096, 32, 8, 14336, 1040), 150, {(6144, 4096): (4, 3)}),
]


@pytest.mark.parametrize("case", range(len(WIDE_EDGES)))
def test_wide_projections_of_uneven_row_groups(case, gemm_plan):
    """Bound: the 16-bit path's 2e-2 logit tolerance, as above."""
    (d, H, Hkv, F, V), n, wide = WIDE_EDGES[case]
    rows, up = -(-n // 64) * 64, lambda x: -(-x // 64) * 64
    part = max((H + 2 * Hkv) * 128, 2 * F, d, up(V)) * max(512, rows)  # the context's room for split sums
    for (N, K), want in wide.items():
        plan = gemm_plan(rows, rows, N, K, 2, min(8, part // (rows * up(N))), part)
        assert (plan.nwn, plan.splits, plan.tile) == (*want, 0), (N, K)
    cfg = di.ModelConfig(f"wide-edge{case}", 1, d, H, Hkv, 128, F, V, dtype="bf16")
    w = di.make_weights(cfg, seed=160 + case, gain_jitter=0.1, threads=16)
    err = _step_error(cfg, w, [7], [n], seed=180 + case)
    print(f"max |logit error| {err:.2e}")
    assert err <= 2e-2


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("n", [1, 2, 64, 65, 256])
def test_a_kept_chain_is_returned_whole(dtype, n):
    """accept(mode=1): the path is the chain, the tokens are those of its nodes after the first and the last node's argmax; for
    the second sequence of a batch too, whose rows start further down."""
    cfg = di.ModelConfig("chain-" + dtype, 1, 128, 1, 1, 128 if dtype == "bf16" else 64, 128, 512, dtype=dtype)
    ver = _verifier(cfg, di.make_weights(cfg, seed=4, gain_jitter=0.1), max_batch=2, kv_capacity=576, max_nodes=max(n, 21))
    prefix = [0, 0]
    for turn, nodes in enumerate(([21, n], [n, 21])):
        tokens = [di.zipf_tokens(cfg.vocab, m, seed=n + turn, stream=b) for b, m in enumerate(nodes)]
        ver.verify_step(prefix, [di.chain_tree(m) for m in nodes], tokens)
        best, _ = ver.get_argmax()
        kept, path, after = ver.accept(mode=1)
        for b, m in enumerate(nodes):
            assert path[b] == list(range(m)) and after[b] == prefix[b] + m
            assert kept[b] == [int(t) for t in tokens[b][1:]] + [int(best[b, m - 1])]
        prefix = after
    ver.close()


# tree sizes, widths: the slim kernel, the stream and wide kernels, the tile kernel (256 and more rows), and the fp32 export
@pytest.mark.parametrize("dtype,nodes,d,V", [("bf16", [3, 9], 128, 1040), ("bf16", [40, 7, 20], 256, 1040), ("bf16", [33, 50], 1024, 8208),
                                             ("bf16", [64, 65, 130], 256, 1040), ("fp32", [5, 17], 128, 101)])
def test_logits_go_to_real_nodes_of_an_array_aligned_to_its_elements(dtype, nodes, d, V):
    """logits_out one element past a 16-byte boundary: real nodes' rows have the bits of the aligned array's, rows of absent nodes and
    what lies before and behind the array keep what was there."""
    import torch
    from paper_2407_12021_amd import binding
    cfg = di.ModelConfig("logits-out-" + dtype, 1, d, 2, 1, 128 if dtype == "bf16" else 64, 256, V, dtype=dtype)
    B, most = len(nodes), max(nodes) + 3
    ver = _verifier(cfg, di.make_weights(cfg, seed=6, gain_jitter=0.1), max_batch=B, kv_capacity=256, max_nodes=most)
    parents = [di.random_tree(n, None, seed=b) for b, n in enumerate(nodes)]
    tokens = [di.zipf_tokens(V, n, seed=6, stream=b) for b, n in enumerate(nodes)]
    want = ver.verify_step([0] * B, parents, tokens, want_logits=True)
    size, mark = B * most * V, 12345.0
    flat = torch.full((size + 64,), mark, device="cuda")
    assert flat.data_ptr() % 16 == 0
    rc = binding.ded_verify_step(ver.ctx, [0] * B, nodes, ver._pad(parents, -1), ver._pad(tokens, 0), flat[1:].data_ptr())
    assert rc == binding.DED_OK
    torch.cuda.synchronize()
    got = flat[1:1 + size].view(B, most, V)
    for b, n in enumerate(nodes):
        assert torch.isfinite(got[b, :n]).all() and torch.equal(got[b, :n], want[b, :n])
        assert (got[b, n:] == mark).all()
    assert flat[0] == mark and (flat[1 + size:] == mark).all()
    ver.close()


def test_a_row_has_the_same_bits_in_a_small_tree_and_a_larger_one():
    """The projections of one and two row blocks add the k ranges of the larger steps in their order: the root's logits of a
    chain of 1, 17 and 40 nodes are equal bit for bit (one key tile each, so attention sums the same keys too)."""
    import torch
    cfg = di.ModelConfig("slim-bits", 2, 4096, 32, 32, 128, 11008, 32000, dtype="bf16")
    w = di.make_weights(cfg, seed=5, gain_jitter=0.1, threads=16)
    ver = _verifier(cfg, w, max_batch=1, kv_capacity=128, max_nodes=40)
    tokens = di.zipf_tokens(cfg.vocab, 60, seed=6)
    ver.verify_step([0], [di.chain_tree(20)], [tokens[:20]])
    ver.accept(mode=1)
    rows = []
    for n in (40, 17, 1):
        rows.append(ver.verify_step([20], [di.chain_tree(n)], [tokens[20:20 + n]], want_logits=True)[0, 0].clone())
    ver.close()
    assert torch.isfinite(rows[0]).all() and rows[0].abs().max() > 0
    assert torch.equal(rows[0], rows[1]) and torch.equal(rows[0], rows[2])


@pytest.mark.parametrize("hd", [8, 16, 64, 128, 256])
def test_fp32_attention_weighs_every_visible_key(hd):
    """A key counts by the mask, not by its score's value: a NaN key of the prefix or of an ancestor reaches the output of
    every row that sees it and of no other, scores of -1e32 are weighed like any others, a score of -infinity weighs nothing.
    Bound for the finite rows: fp32 sums of at most 41 values of O(1), 1e-5."""
    import torch
    P, n, cap = 37, 4, 64
    cfg = di.ModelConfig(f"f32-attn{hd}", 1, 64, 2, 1, hd, 64, 64, dtype="fp32")
    ver = _verifier(cfg, di.make_weights(cfg, seed=3), max_batch=1, kv_capacity=cap, max_nodes=n)
    g = torch.Generator(device="cuda").manual_seed(hd)
    rand = lambda *shape: torch.randn(*shape, device="cuda", generator=g)
    k, v = rand(1, P, hd), rand(1, P, hd)
    q, kt, vt = rand(1, n, 2, hd), rand(1, 1, n, hd), rand(1, 1, n, hd)
    parent = [-1, 0, 0, 1]
    sees = np.array([[1, 0, 0, 0], [1, 1, 0, 0], [1, 0, 1, 0], [1, 1, 0, 1]], bool)

    def run(k, q, kt):
        ver.kv_store(0, 0, 0, k, v)
        return ver.tree_attention(0, [P], [parent], q, kt, vt)[0].cpu().numpy().astype(np.float64)

    def ref(k, q, kt):
        K, V = (torch.cat([a[0], b[0, 0]]).double().cpu().numpy() for a, b in ((k, kt), (v, vt)))
        out = np.zeros((n, 2, hd))
        for i in range(n):
            see = np.concatenate([np.ones(P, bool), sees[i]])
            for h in range(2):
                s = K[see] @ q[0, i, h].double().cpu().numpy() / np.sqrt(hd)
                w = np.exp(s - s.max())
                out[i, h] = w @ V[see] / w.sum()
        return out

    assert np.abs(run(k, q, kt) - ref(k, q, kt)).max() <= 1e-5
    for at in (0, 15, 36):
        bad = k.clone()
        bad[0, at, hd // 2] = float("nan")
        assert np.isnan(run(bad, q, kt)).all(), at
    bad = kt.clone()
    bad[0, 0, 1, 3] = float("nan")
    out = run(k, q, bad)
    assert np.isnan(out[[1, 3]]).all() and np.abs(out[[0, 2]] - ref(k, q, kt)[[0, 2]]).max() <= 1e-5
    # every visible score below -1e32, two keys tied at the top
    ones, far = torch.ones_like(q), torch.full_like(k, -4e32 / hd ** 0.5)
    far[0, [2, 30]] /= 2
    far_t = torch.full_like(kt, -4e32 / hd ** 0.5)
    assert np.abs(run(far, ones, far_t) - ref(far, ones, far_t)).max() <= 1e-5
    gone = k.clone()
    gone[0, :33, 0] = float("-inf")
    assert np.abs(run(gone, ones, kt) - ref(gone, ones, kt)).max() <= 1e-5
    ver.close()


def test_fp32_step_reports_a_nan_key_of_the_prefix():
    """A restored prefix with one bad key and finite values: no tokens, an error."""
    from paper_2407_12021_amd.binding import DED_ENONFINITE, DedError
    cfg = di.ModelConfig("f32-nan-key", 2, 64, 2, 1, 32, 64, 96, dtype="fp32")
    ver = _verifier(cfg, di.make_weights(cfg, seed=3), max_batch=1, kv_capacity=64, max_nodes=16)
    r = np.random.default_rng(2)
    k, v = (r.standard_normal((1, 20, 32)).astype(np.float32) for _ in range(2))
    for bad in (False, True):
        k[0, 7, 5] = np.nan if bad else 0.5
        for layer in range(2):
            ver.kv_store(layer, 0, 0, k, v)
        ver.verify_step([20], [di.random_tree(9, None, seed=1)], [di.zipf_tokens(96, 9, seed=1)])
        if not bad:
            ver.accept(mode=0)
            continue
        for call in (ver.get_argmax, ver.accept):
            with pytest.raises(DedError) as e:
                call()
            assert e.value.code == DED_ENONFINITE
    ver.close()


# (d, H, Hkv, F, V) of one layer; a batch of full trees and a ragged one that share the first tree.  320 padded rows whose
# gate / up slices have no room in the context where those of the 208 packed rows would; 192 and 144 padded rows, whose QKV
# or gate / up run in the tile kernel beside full trees and in the wide kernel (128 packed rows) beside small ones, the LM
# head in two shapes of tile; 512 padded rows beside 192 and 384 packed ones, which between them take every shape of tile
RAGGED = [
    ((4096, 32, 32, 11008, 32000), [64] * 5, [64, 33, 16, 20, 40]),
    ((4096, 32, 32, 11008, 32000), [64] * 3, [64, 16, 17]),
    ((4096, 32, 8, 14336, 32000), [48] * 3, [48, 16, 1]),
    ((4096, 32, 8, 14336, 32000), [64] * 8, [64] + [16] * 7),
    ((4096, 32, 8, 14336, 32000), [64] * 8, [64] * 4 + [32] * 4),
]


@pytest.mark.parametrize("case", range(len(RAGGED)))
def test_a_tree_has_the_same_bits_beside_full_trees_and_beside_small_ones(case):
    """The k ranges of a product come from the trees padded to the largest, whatever runs: the logits of the first tree do
    not depend on how far its neighbours fall short of it."""
    import torch
    (d, H, Hkv, F, V), full, ragged = RAGGED[case]
    cfg = di.ModelConfig(f"ragged-bits{case}", 1, d, H, Hkv, 128, F, V, dtype="bf16")
    w = di.make_weights(cfg, seed=5, gain_jitter=0.1, threads=16)
    ver = _verifier(cfg, w, max_batch=len(full), kv_capacity=128, max_nodes=max(full))
    r = np.random.default_rng(7)
    k, v = (torch.from_numpy(r.standard_normal((Hkv, 20, 128)).astype(np.float32)).bfloat16() for _ in range(2))
    rows = []
    for nodes in (full, ragged):
        for b in range(len(nodes)):
            ver.kv_store(0, b, 0, k, v)
        parents = [di.random_tree(n, None, seed=b) for b, n in enumerate(nodes)]
        tokens = [di.zipf_tokens(V, n, seed=6, stream=b) for b, n in enumerate(nodes)]
        rows.append(ver.verify_step([20] * len(nodes), parents, tokens, want_logits=True)[0].clone())
    ver.close()
    assert torch.isfinite(rows[0]).all() and rows[0].abs().max() > 0
    assert torch.equal(rows[0], rows[1])


def test_cache_copies_are_done_for_every_stream():
    """The tensors of kv_store and kv_load are used on another stream right after the call, behind a long queue of work on
    the context's own."""
    import torch
    cfg = di.ModelConfig("kv-streams", 1, 128, 4, 2, 128, 128, 64, dtype="bf16")
    ver = _verifier(cfg, di.make_weights(cfg, seed=3), max_batch=1, kv_capacity=4096, max_nodes=16)
    other = torch.cuda.Stream()
    a = torch.randn(2, 4000, 128, device="cuda").bfloat16().clamp(0.5, 4.0)
    busy = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    staging = a.clone()
    for _ in range(20):
        busy @ busy
    ver.kv_store(0, 0, 0, staging, staging)
    with torch.cuda.stream(other):
        staging.zero_()
    for _ in range(20):
        busy @ busy
    k, v = ver.kv_load(0, 0, 0, 4000)
    with torch.cuda.stream(other):
        same = torch.equal(k, a) and torch.equal(v, a)
    assert same
    ver.close()


def _off_by_one(x):
    """The same values one element past an allocation's start."""
    import torch
    y = torch.empty(x.numel() + 1, dtype=x.dtype, device=x.device)[1:].view(x.shape)
    y.copy_(x)
    return y


@pytest.mark.parametrize("dtype,prefix,n", [("bf16", 40, 16), ("bf16", 1500, 40), ("fp32", 40, 16)])
def test_rows_of_a_caller_are_aligned_to_their_elements_only(dtype, prefix, n, monkeypatch):
    """Queries, tree K/V, output and plain cache rows (fp32: the cache itself too) that start one element past a 16-byte
    boundary give the bits of aligned ones, with one key range and with several."""
    import torch
    from paper_2407_12021_amd import binding
    hd = 128 if dtype == "bf16" else 64
    cfg = di.ModelConfig("align-" + dtype, 1, 128, 4, 2, hd, 128, 64, dtype=dtype)
    w = di.make_weights(cfg, seed=3)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(n)
    rand = lambda *shape: torch.randn(*shape, device="cuda", generator=g).to(dt)
    k, v, q = rand(2, prefix, hd), rand(2, prefix, hd), rand(1, n, 4, hd)
    kt, vt = rand(1, 2, n, hd), rand(1, 2, n, hd)
    parent, token = di.random_tree(n, None, seed=n), di.zipf_tokens(64, n, seed=n)
    got = []
    for shift in (lambda x: x, _off_by_one):
        if dtype == "fp32" and shift is _off_by_one:
            init, size = binding.ded_verify_init, binding.ded_kv_layer_bytes

            def init_off(cfg, weights, kv, *rest):
                kv.k[0] += 4
                kv.v[0] += 4
                return init(cfg, weights, kv, *rest)

            monkeypatch.setattr(binding, "ded_kv_layer_bytes", lambda c: size(c) + 4)
            monkeypatch.setattr(binding, "ded_verify_init", init_off)
        ver = _verifier(cfg, w, max_batch=1, kv_capacity=prefix + 64, max_nodes=n)
        ver.kv_store(0, 0, 0, shift(k), shift(v))
        out = ver.tree_attention(0, [prefix], [parent], shift(q), shift(kt), shift(vt), out=shift(torch.zeros_like(q)))
        lk, lv = shift(torch.zeros_like(k)), shift(torch.zeros_like(v))
        assert binding.ded_kv_load(ver.ctx, 0, 0, 0, prefix, lk.data_ptr(), lv.data_ptr()) == binding.DED_OK
        logits = ver.verify_step([prefix], [parent], [token], want_logits=True)
        torch.cuda.synchronize()
        got.append([x.clone() for x in (out, lk, lv, logits)])
        ver.close()
    for a, b in zip(*got):
        assert a.any() and torch.equal(a, b)


@pytest.mark.parametrize("dtype,max_nodes", [("bf16", 33), ("fp32", 33), ("bf16", 256)])
def test_calls_in_a_row_keep_their_own_descriptions(dtype, max_nodes):
    """Forty attention calls and ten steps that nobody waits for in between, each with its own tree and prefix length (more calls
    than the pinned mirror has slots): every output has the bits of the same call waited for."""
    import torch
    hd, batch = 128 if dtype == "bf16" else 64, 2
    cfg = di.ModelConfig("in-a-row-" + dtype, 1, 128, 4, 2, hd, 256, 96, dtype=dtype)
    ver = _verifier(cfg, di.make_weights(cfg, seed=3), max_batch=batch, kv_capacity=640, max_nodes=max_nodes)
    kind = torch.bfloat16 if dtype == "bf16" else torch.float32
    draw = lambda *shape: torch.randn(*shape, device="cuda").to(kind)
    for b in range(batch):
        ver.kv_store(0, b, 0, draw(2, 300, hd), draw(2, 300, hd))
    r = np.random.default_rng(11)
    calls = []
    for i in range(50):
        nodes = [int(r.integers(1, max_nodes + 1)) for _ in range(batch)]
        calls.append(([int(r.integers(0, 301)) for _ in nodes], [di.random_tree(n, None, seed=i) for n in nodes],
                      draw(batch, max_nodes, 4, hd), draw(batch, 2, max_nodes, hd), draw(batch, 2, max_nodes, hd),
                      [di.zipf_tokens(96, n, seed=i, stream=b) for b, n in enumerate(nodes)]))
    runs = []
    for wait in (True, False):
        for b in range(batch):
            k = torch.linspace(-1, 1, 2 * 300 * hd, device="cuda").view(2, 300, hd).to(kind)
            ver.kv_store(0, b, 0, k, k.flip(1).contiguous())
        outs = []
        for i, (prefix, parents, q, k, v, tokens) in enumerate(calls):
            if i % 5:
                outs.append(ver.tree_attention(0, prefix, parents, q, k, v))
            else:
                outs.append(ver.verify_step(prefix, parents, tokens, want_logits=True))
            if wait:
                torch.cuda.synchronize()
        torch.cuda.synchronize()
        runs.append(outs)
    ver.close()
    for i, (a, b) in enumerate(zip(*runs)):
        assert torch.isfinite(a).all() and torch.equal(a, b), i


@pytest.mark.parametrize("batch", [8, 9])
def test_attention_of_up_to_eight_sequences_and_more(batch):
    """Up to eight sequences' places travel with the scatter's launch, more are read from the step's description: every tree's keys and
    values land in its own slots.  Bound: bf16 outputs of O(1), 2^-9, and f16 weights, together under 2e-2."""
    import torch
    H, Hkv, most = 2, 1, 20
    cfg = di.ModelConfig(f"scatter{batch}", 1, 128, H, Hkv, 128, 128, 64, dtype="bf16")
    ver = _verifier(cfg, di.make_weights(cfg, seed=3), max_batch=batch, kv_capacity=192, max_nodes=most)
    g = torch.Generator(device="cuda").manual_seed(batch)
    draw = lambda *shape: torch.randn(*shape, device="cuda", generator=g).bfloat16()
    prefix, nodes = [7 * b for b in range(batch)], [1 + (5 * b) % most for b in range(batch)]
    parents = [di.random_tree(n, None, seed=b) for b, n in enumerate(nodes)]
    kp, vp = draw(batch, Hkv, 64, 128), draw(batch, Hkv, 64, 128)
    q, kt, vt = draw(batch, most, H, 128), draw(batch, Hkv, most, 128), draw(batch, Hkv, most, 128)
    for b, p in enumerate(prefix):
        if p:
            ver.kv_store(0, b, 0, kp[b, :, :p].contiguous(), vp[b, :, :p].contiguous())
    out = ver.tree_attention(0, prefix, parents, q, kt, vt)
    for b, (p, n) in enumerate(zip(prefix, nodes)):
        k, v = ver.kv_load(0, b, 0, p + n)
        assert torch.equal(k[:, p:], kt[b, :, :n]) and torch.equal(v[:, p:], vt[b, :, :n]), b
        kk, vv = (torch.cat([a[b, :, :p], t[b, :, :n]], 1).transpose(0, 1).double().cpu().numpy() for a, t in ((kp, kt), (vp, vt)))
        vis = np.concatenate([np.ones((n, p), bool), oracle.ancestor_mask(parents[b])], axis=1)
        ref = oracle.masked_attention(q[b, :n].double().cpu().numpy(), kk, vv, vis)
        assert np.abs(out[b, :n].double().cpu().numpy() - ref).max() <= 2e-2, b
    ver.close()
