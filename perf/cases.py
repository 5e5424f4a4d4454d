"""Performance cases of the library: what a program that prunes a KV cache during prefill asks of it.

Five kinds of call, each through the public entry points:
  layer  one layer's step (score, centrality update, selection, cache store): sweep.LayerSweep.layer
  pivot  one layer scored together with the pivot detector's metrics: sweep.LayerSweep.score_pivot
  sweep  all layers of a prefill on four streams, then the propagation indices: LayerSweep.sweep_chains
  prune  the structural truncation: top-k of the centrality, hidden rows and positions of the kept tokens
  paged  a paged cache's eviction: block scores, top-k of the blocks, gather of the kept blocks' K and V

Inputs are N(0, 1) queries, keys and values in which as many keys as the budget holds are heavy hitters, aligned
with their KV group's mean query (4 sqrt(head_dim) along it, as the repository's synthetic workloads plant their
hubs).  The kept set is then separated from the rest by far more than rounding, so indices and caches are
comparable entry by entry.
"""
import math

import torch

from paper_2604_06746_amd import binding as B
from paper_2604_06746_amd.sweep import LayerSweep

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(kind, name=None, *, heads=32, kv_heads=8, head_dim=128, window=64, dtype="bf16", causal=False, lengths="131072",
          keep=0.03125, layers=1, hidden=0, block=0):
    c = dict(kind=kind, heads=heads, kv_heads=kv_heads, head_dim=head_dim, window=window, dtype=dtype, causal=causal,
             lengths=lengths, keep=keep, layers=layers, hidden=hidden, block=block)
    return dict(c, name=name) if name else c


# eight prompts of 16K to 128K tokens (the repository's ragged batch configuration)
RAGGED8 = "73146,32809,34880,88336,113661,94010,18829,79122"


def listed():
    return [
        # the smallest prefill, full precision, one KV head per query head: launches and latency
        _case("layer", "layer_f32_1k", heads=8, kv_heads=8, head_dim=64, window=32, dtype="f32", lengths="1024", keep=0.125),
        # a few short prompts batched together, causal, with the method's own window of 8
        _case("layer", "layer_short_ragged_w8_causal", window=8, causal=True, lengths="700,33,1500,64", keep=0.05),
        # the method's own operating point: 32K tokens, window 8, 10 % budget
        _case("layer", "layer_32k_w8", window=8, lengths="32768", keep=0.1),
        # a 32K-token prefill with a window of 32
        _case("layer", "layer_32k_w32", window=32, lengths="32768", keep=0.0625),
        # one layer of the headline configuration
        _case("layer", "layer_128k_w64", lengths="131072", keep=0.03125),
        # a ragged batch of long prompts: odd lengths, K streamed from HBM
        _case("layer", "layer_ragged8_w32", window=32, lengths=RAGGED8, keep=0.05),
        # the longest context
        _case("layer", "layer_1m_w64", lengths="1048576", keep=0.015625),
        # layers on which the pivot detector runs: at the method's operating point and at the headline's size
        _case("pivot", "pivot_32k_w8", window=8, lengths="32768", keep=0.1),
        _case("pivot", "pivot_128k_w64", lengths="131072", keep=0.03125),
        # the headline: every layer of a 128K-token prefill
        _case("sweep", "sweep_128k_w64", lengths="131072", keep=0.03125, layers=32),
        # the pivot layer's truncation of the hidden states to 20 %
        _case("prune", "prune_128k", lengths="131072", keep=0.2, hidden=4096),
        # eviction from a paged cache, blocks of 16 tokens
        _case("paged", "paged_128k_b16", lengths="131072", keep=0.1, block=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cut(rng, total, parts, least):
    """`parts` ragged lengths that add up to about `total`, none below `least`."""
    w = [rng.uniform(0.2, 1.0) for _ in range(parts)]
    return [max(least, int(total * x / sum(w))) for x in w]


def draw(rng):
    kind = rng.choices(("layer", "f32", "pivot", "sweep", "prune", "paged"), (9, 2, 3, 2, 2, 2))[0]
    heads, kv_heads, head_dim = rng.choice(((32, 8, 128), (32, 8, 128), (8, 2, 128), (16, 2, 128), (32, 32, 128), (8, 8, 64), (32, 8, 64)))
    window = rng.choice((8, 16, 32, 32, 64, 64))
    keep = rng.choice((0.015625, 0.03125, 0.05, 0.1, 0.2))
    causal = rng.random() < 0.3
    # a context costs what its keys and its query rows cost: keep both below the largest listed cases
    top = min(1048576, 1048576 * 8 * 128 // max(kv_heads * head_dim, 8 * 128 * heads * window // 2048))
    if causal and window % 32:
        top = min(top, 131072)
    if kind == "f32":
        lengths = _cut(rng, _log(rng, 256, 8192), rng.choice((1, 1, 3)), window + 4)
        return _case("layer", heads=heads, kv_heads=kv_heads, head_dim=head_dim, window=window, dtype="f32", causal=causal,
                     lengths=",".join(map(str, lengths)), keep=keep)
    if kind == "layer":
        parts = rng.choice((1, 1, 2, 5, 8, 17))
        lengths = _cut(rng, _log(rng, 1024, top), parts, window + 4)
        return _case("layer", heads=heads, kv_heads=kv_heads, head_dim=head_dim, window=window, causal=causal,
                     lengths=",".join(map(str, lengths)), keep=keep)
    if kind == "pivot":
        lengths = _cut(rng, _log(rng, 2048, 131072), rng.choice((1, 1, 2)), 512)
        return _case("pivot", heads=heads, kv_heads=kv_heads, head_dim=head_dim, window=window, causal=causal,
                     lengths=",".join(map(str, lengths)), keep=keep)
    if kind == "sweep":
        return _case("sweep", window=window, lengths=str(_log(rng, 4096, 98304)), keep=min(keep, 0.1), layers=rng.choice((6, 13, 32)))
    if kind == "prune":
        lengths = _cut(rng, _log(rng, 4096, 131072), rng.choice((1, 1, 4)), window + 4)
        return _case("prune", window=window, lengths=",".join(map(str, lengths)), keep=rng.choice((0.1, 0.2, 0.6)),
                     hidden=rng.choice((1024, 4096, 5120)))
    block = rng.choice((16, 32, 64))
    blocks = max(64, _log(rng, 4096, 524288) // block)
    return _case("paged", kv_heads=kv_heads, head_dim=head_dim, window=window, lengths=str(block * blocks), keep=keep, block=block)


def _sizes(case):
    lengths = [int(x) for x in case["lengths"].split(",")]
    budgets = [min(int(case["keep"] * n), n - case["window"]) for n in lengths]
    return lengths, budgets


def _gen(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + tag)
    return g


def _scores(n, g):
    """Skewed positive scores, as an accumulated centrality has them."""
    return torch.exp(0.5 * torch.randn(n, generator=g, device="cuda")) / n


def _layer_inputs(case, seed, layer):
    """(q_win [B, heads, window, head_dim], k, v [kv_heads, tokens, head_dim]) with heavy hitters as above."""
    lengths, budgets = _sizes(case)
    H, G, d, w, dt = case["heads"], case["kv_heads"], case["head_dim"], case["window"], DTYPES[case["dtype"]]
    g = _gen(seed, layer)
    q = torch.randn(len(lengths), H, w, d, generator=g, device="cuda", dtype=dt)
    k = torch.randn(G, sum(lengths), d, generator=g, device="cuda", dtype=dt)
    v = torch.randn(G, sum(lengths), d, generator=g, device="cuda", dtype=dt)
    mean = q.float().reshape(len(lengths), G, -1, d).mean(dim=2)
    along = 4.0 * math.sqrt(d) * mean / mean.norm(dim=2, keepdim=True)
    lo = 0
    for b, (n, hitters) in enumerate(zip(lengths, budgets)):
        at = lo + torch.randperm(n - w, generator=g, device="cuda")[:hitters]
        k[:, at] = (k[:, at].float() + along[b][:, None, :]).to(dt)
        lo += n
    return q, k, v


def prepare(case, seed):
    lengths, budgets = _sizes(case)
    cu = [0]
    for n in lengths:
        cu.append(cu[-1] + n)
    s = dict(kind=case["kind"], cu=cu, budgets=budgets, window=case["window"])
    if case["kind"] == "prune":
        g = _gen(seed, 1)
        s["rows"] = [k + case["window"] for k in budgets]
        s["scores"] = _scores(cu[-1], g)
        s["hidden"] = torch.randn(cu[-1], case["hidden"], generator=g, device="cuda", dtype=torch.bfloat16)
        s["positions"] = torch.cat([torch.arange(n, device="cuda") for n in lengths])
        s["idx"] = torch.empty(sum(s["rows"]), dtype=torch.int32, device="cuda")
        s["hidden_out"] = torch.empty(sum(s["rows"]), case["hidden"], device="cuda", dtype=torch.bfloat16)
        s["positions_out"] = torch.empty(sum(s["rows"]), dtype=torch.int64, device="cuda")
        s["workspace"] = torch.empty(B.structkv_workspace_bytes(None, len(lengths), cu[-1]), dtype=torch.uint8, device="cuda")
        return s
    if case["kind"] == "paged":
        g = _gen(seed, 2)
        n, block, G, d = cu[-1], case["block"], case["kv_heads"], case["head_dim"]
        blocks, tail = n // block, -(-case["window"] // block)
        kept = min(int(case["keep"] * blocks), blocks - tail)
        s.update(block=block, block_cu=[0, blocks], kept=[kept], tail=tail, rows=[kept + tail])
        s["scores"] = _scores(n, g)
        s["k"], s["v"] = (torch.randn(G, blocks, block * d, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        s["block_scores"] = torch.empty(blocks, device="cuda")
        s["idx"] = torch.empty(kept + tail, dtype=torch.int32, device="cuda")
        s["k_out"], s["v_out"] = (torch.empty(G, kept + tail, block * d, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        s["workspace"] = torch.empty(B.structkv_workspace_bytes(None, 1, blocks), dtype=torch.uint8, device="cuda")
        return s
    s["sweep"] = LayerSweep(case["heads"], case["kv_heads"], case["head_dim"], case["window"], DTYPES[case["dtype"]], lengths,
                            budgets, causal=case["causal"], n_layers_out=case["layers"])
    s["layers"] = [_layer_inputs(case, seed, layer) for layer in range(case["layers"])]
    if case["kind"] == "sweep":
        s["streams"] = [torch.cuda.Stream() for _ in range(3)]
    return s


def run(s):
    if s["kind"] == "prune":
        B.structkv_select_topk(s["scores"], s["cu"], s["budgets"], s["window"], s["idx"], s["workspace"])
        B.structkv_truncate_hidden(s["hidden"], s["hidden_out"], s["positions"], s["positions_out"], s["cu"], s["rows"], s["idx"])
        return [s["idx"], s["hidden_out"], s["positions_out"]]
    if s["kind"] == "paged":
        B.structkv_block_scores(s["scores"], s["cu"], s["block"], s["block_scores"])
        B.structkv_select_topk(s["block_scores"], s["block_cu"], s["kept"], s["tail"], s["idx"], s["workspace"])
        B.structkv_gather_kv(s["k"], s["v"], s["k_out"], s["v_out"], s["block_cu"], s["rows"], s["idx"])
        return [s["block_scores"], s["idx"], s["k_out"], s["v_out"]]
    sw = s["sweep"]
    if s["kind"] == "pivot":
        q, k, _ = s["layers"][0]
        sparsity, variance = sw.score_pivot(q, k)
        return [sw.indeg, sw.entropy, sw.entropy_per_head, sparsity, variance]
    if s["kind"] == "layer":
        q, k, v = s["layers"][0]
        sw.layer(q, k, v)
        return [sw.indeg, sw.centrality, sw.entropy, sw.entropy_per_head, sw.idx_kv, sw.k_cache, sw.v_cache]
    sw.reset()
    sw.sweep_chains(s["layers"], s["streams"])
    sw.select_struct()
    return [sw.indeg, sw.centrality, sw.entropy, sw.entropy_per_head, sw.idx_kv, sw.idx_struct, sw.k_cache, sw.v_cache]


def work(case):
    lengths, budgets = _sizes(case)
    n, e = sum(lengths), 4 if case["dtype"] == "f32" else 2
    rows = sum(budgets) + case["window"] * len(lengths)
    if case["kind"] == "prune":   # scores; kept hidden rows and positions in and out; indices
        return {"bytes": 4 * n + rows * (2 * 2 * case["hidden"] + 2 * 8 + 4), "flops": 0}
    if case["kind"] == "paged":   # scores; block scores; kept K and V blocks in and out; indices
        blocks, tail = n // case["block"], -(-case["window"] // case["block"])
        kept = min(int(case["keep"] * blocks), blocks - tail) + tail
        return {"bytes": 4 * n + 4 * blocks + kept * (2 * 2 * 2 * case["kv_heads"] * case["block"] * case["head_dim"] + 4), "flops": n}
    # window queries and keys in; in-degrees out; entropies out; one contraction of the window with all keys
    q = len(lengths) * case["heads"] * case["window"] * case["head_dim"] * e
    k = n * case["kv_heads"] * case["head_dim"] * e
    moved = q + k + 4 * n + 4 * len(lengths) * (1 + case["heads"])
    flops = 2 * case["heads"] * case["window"] * case["head_dim"] * n
    if case["kind"] != "pivot":   # centrality in and out; kept K and V rows in and out; indices
        moved += 2 * 4 * n + rows * (2 * 2 * case["kv_heads"] * case["head_dim"] * e + 4)
    return {"bytes": moved * case["layers"], "flops": flops * case["layers"]}


def tolerance(case):
    if case["kind"] in ("prune", "paged"):   # selections and copies; block sums are added left to right by contract
        return "exact"
    return {"rel": 4e-6, "max": 1e-5, "differ": 0.0}   # four to five times what the path differs by from 64 bits
