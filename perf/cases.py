"""Timed workloads of the SharePrefill attention library: what a prefill asks of its public entry points.

Inputs are the synthetic prompts of synth/generator.py in torch on the GPU: per head cluster a piecewise-constant topic
sequence that lifts the logits of query / key pairs of one topic, a sink key at token 0, a few heavy vertical keys and
i.i.d. N(0,1) noise.  `spread` gives the heads of a cluster different sparsities, so that the thresholds of the gate
(Alg. 3) split them into pivots, sharing heads and heads that fall back.

A case is a dict:
  kind        layer   one fused layer (sp_prefill_layer), score maps returned when `scores`
              printed the pattern construction as the paper prints it (sp_prefill_layer_modes, mean logits + one
                      selection over the flattened map), score maps kept in the workspace
              gated   a fused layer behind Alg. 3's gate (sp_prefill_layer_gated)
              stack   `layers` layers of one prompt through the pattern dictionary (sp_prefill_layer_dict)
              slash   attention over the vertical-slash pattern, token by token (sp_vertical_slash_attn)
              dense   dense attention on every head with its score maps (sp_dense_attn_with_block_scores)
              lists   block-sparse attention over the caller's lists (sp_block_sparse_attn): sink, window, verticals
  batch, seq, q_heads, kv_heads, head_dim, block, cluster (heads per cluster), gamma
"""
import math

import numpy as np
import torch

import paper_2505_19578_amd as sp


def _case(name, kind, seq, q_heads=32, kv_heads=8, head_dim=128, block=128, cluster=4, gamma=0.95, batch=1, **more):
    c = {"kind": kind, "batch": batch, "seq": seq, "q_heads": q_heads, "kv_heads": kv_heads, "head_dim": head_dim,
         "block": block, "cluster": cluster, "gamma": gamma}
    c.update(more)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: the tiny configuration, where launches and latency are what a user waits for
        _case("tiny_1k", "layer", 1024, 4, 4, 64, 64, 2, 0.9, mixed=False, scores=True),
        # a chat turn: the Llama-3-8B shape on a short prompt
        _case("layer_4k", "layer", 4096, mixed=False, scores=False),
        # a document: the 32K configuration
        _case("layer_32k", "layer", 32768, mixed=False, scores=True),
        # the headline configuration
        _case("layer_128k", "layer", 131072, mixed=False, scores=True),
        # the printed construction on the Qwen2.5-7B shape: clusters straddle KV heads, a length of 193 blocks
        _case("printed_24k", "printed", 24704, 28, 4, gamma=0.9, mixed=True),
        # two prompts in one call in the finer blocks of 64, roles decided on the device at the paper's thresholds
        _case("gated_8k_batch2", "gated", 8128, block=64, gamma=0.9, batch=2, mixed=False, spread=True, delta=0.3, tau=0.2),
        # a prefill at the paper's thresholds: pivots, sharing heads and token-level fallback, 313 blocks
        _case("stack_40k", "stack", 40064, gamma=0.9, mixed=False, spread=True, layers=4, delta=0.3, tau=0.2,
              fallback="tokens"),
        # a prefill without the sparsity exclusion: one layer with pivots, then every head shares a pattern
        _case("stack_open_64k", "stack", 65536, mixed=False, spread=False, layers=4, delta=10.0, tau=0.2,
              fallback="dense"),
        # every head falls back: a short prompt, and the longest
        _case("slash_8k", "slash", 8192, gamma=0.9, mixed=False),
        _case("slash_128k", "slash", 131072, mixed=False),
        # score maps of every head for the offline clustering of heads: head_dim 64, blocks of 64, odd length
        _case("dense_12k_d64", "dense", 12352, 16, 16, 64, 64, batch=2, mixed=False),
        # the Llama-3.1-70B shape over lists that the caller made
        _case("lists_96k", "lists", 98304, 64, 8, mixed=False),
    ]


_KINDS = ["layer", "layer", "printed", "gated", "stack", "slash", "dense", "lists"]
# query heads, KV heads, head_dim, block, heads per cluster
_SHAPES = [(32, 8, 128, 128, 4), (28, 4, 128, 128, 4), (64, 8, 128, 128, 4), (32, 8, 128, 64, 4), (16, 16, 64, 64, 4),
           (4, 4, 64, 64, 2), (32, 8, 64, 128, 4)]


def draw(rng):
    """One more case: any kind and shape, the length spread over its logarithm, in whole blocks: from 1K to 128K, with
    the finer blocks of 64 (whose maps are four times as large) to 16K."""
    kind = rng.choice(_KINDS)
    q_heads, kv_heads, head_dim, block, cluster = rng.choice(_SHAPES)
    blocks = round(math.exp(rng.uniform(math.log(1024), math.log(131072 if block == 128 else 16384))) / block)
    c = _case(None, kind, blocks * block, q_heads, kv_heads, head_dim, block, cluster, rng.choice([0.9, 0.95]),
              rng.choice([1, 1, 1, 2]), mixed=rng.random() < 0.3)
    if kind == "layer":
        c["scores"] = rng.random() < 0.5
    if kind in ("gated", "stack"):
        c["spread"] = rng.random() < 0.7
        c["delta"], c["tau"] = rng.choice([(0.3, 0.2), (10.0, 0.2)])
    if kind == "stack":
        c["layers"] = rng.choice([2, 3, 4])
        c["fallback"] = rng.choice(["tokens", "tokens", "blocks", "dense"])
    most = 0.8 * max(_pairs(x) * x["head_dim"] for x in listed())
    while _pairs(c) * c["head_dim"] > most:
        c["seq"] = max(8, int(c["seq"] // block * 0.7)) * block
    return c


# ------------------------------------------------------------------------------------------------ inputs
def _rand(seed, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _clusters(c, rng):
    size, heads = c["cluster"], c["q_heads"]
    order = rng.permutation(heads) if c["mixed"] else np.arange(heads)
    h2c = [0] * heads
    for at, h in enumerate(order):
        h2c[int(h)] = at // size
    pivots = [min(h for h in range(heads) if h2c[h] == x) for x in range(heads // size)]
    return h2c, pivots


def _prompt(c, seed):
    """What the layers of one prompt have in common: topics per cluster, heavy positions."""
    rng = np.random.default_rng([seed, 1])
    n, block, rank = c["seq"], c["block"], 4 if c["seq"] <= 1024 else 8
    topics = []
    for _ in range(c["q_heads"] // c["cluster"]):
        t, at = np.empty(n, dtype=np.int64), 0
        while at < n:
            seg = int(rng.integers(2 * block, 16 * block + 1))
            t[at:at + seg] = int(rng.integers(0, rank))
            at += seg
        topics.append(torch.from_numpy(t).cuda())
    heavy = rng.choice(np.arange(1, n), size=16, replace=False) if n > 1024 else np.zeros(0, dtype=np.int64)
    return topics, rank, torch.from_numpy(heavy).cuda()


# per head of a cluster: how strongly its queries follow the topics, and by how many topics it is shifted (one head in
# four is far from its cluster: highly sparse in one cluster, on other topics in the next)
_SPREAD_GAIN = (0.04, 0.05, 0.04, 0.045, 0.04, 0.05, 0.04, 1.0)
_SPREAD_SHIFT = (0, 0, 0, 3, 0, 0, 0, 0)


def _layer_inputs(c, h2c, prompts, seed):
    """q, k, v of one layer, bf16 [batch][seq][heads][head_dim]."""
    n, d, heads, kv = c["seq"], c["head_dim"], c["q_heads"], c["kv_heads"]
    q = torch.empty((c["batch"], n, heads, d), dtype=torch.bfloat16, device="cuda")
    k = torch.empty((c["batch"], n, kv, d), dtype=torch.bfloat16, device="cuda")
    v = torch.empty_like(k)
    gain = math.sqrt(6.0 * math.sqrt(d))
    rank_in = [sum(1 for x in range(h) if h2c[x] == h2c[h]) for h in range(heads)]
    for b, (topics, rank, heavy) in enumerate(prompts):
        s = (seed * 1009 + b) * 4096
        proj = _rand(s, len(topics), rank, d) / math.sqrt(d)
        proj_v = _rand(s + 1, len(topics), rank, d) / math.sqrt(d)
        sink = torch.nn.functional.normalize(_rand(s + 2, d), dim=0)
        boost = torch.zeros(n, device="cuda")
        boost[0] = 4.0
        boost[heavy] = 10.0
        for h in range(heads):
            at = h2c[h] * c["cluster"] + rank_in[h]
            follow, shift = (_SPREAD_GAIN[at % 8], _SPREAD_SHIFT[at % 8]) if c.get("spread") else (1.0, 0)
            own = proj[h2c[h]] * (gain * math.sqrt(follow)) + 4.0 * sink
            q[b, :, h] = _rand(s + 8 + h, n, d) + own[(topics[h2c[h]] + shift) % rank]
        for g in range(kv):
            x, y = _rand(s + 1024 + g, n, d), _rand(s + 2048 + g, n, d)
            for cl in sorted({h2c[h] for h in range(g * heads // kv, (g + 1) * heads // kv)}):
                x += (gain * proj[cl])[topics[cl]]
                y += (4.0 * proj_v[cl])[topics[cl]]
            k[b, :, g] = x + boost[:, None] * (math.sqrt(d) / 4.0) * sink
            v[b, :, g] = y
    return q, k, v


def _caller_lists(c, rng):
    """Lists of n maps: the sink block, a window below the query block and a few vertical block columns."""
    nqb, maps = c["seq"] // c["block"], max(1, c["q_heads"] // 4)
    i, j = torch.arange(nqb, device="cuda")[:, None], torch.arange(nqb, device="cuda")[None, :]
    idx = torch.full((c["batch"], maps, nqb, nqb), -1, dtype=torch.int32, device="cuda")
    cnt = torch.empty((c["batch"], maps, nqb), dtype=torch.int32, device="cuda")
    for b in range(c["batch"]):
        for m in range(maps):
            column = torch.zeros(nqb, dtype=torch.bool, device="cuda")
            column[torch.from_numpy(rng.choice(nqb, size=max(1, nqb // 12), replace=False)).cuda()] = True
            column[0] = True
            keep = (column[None, :] | (i - j < int(rng.integers(8, 33)))) & (j <= i)
            key = torch.where(keep, j, nqb).sort(dim=1).values
            idx[b, m] = torch.where(key < nqb, key, -1).to(torch.int32)
            cnt[b, m] = keep.sum(dim=1, dtype=torch.int32)
    return idx, cnt, maps


def prepare(case, seed):
    c, kind = case, case["kind"]
    rng = np.random.default_rng([seed, 2])
    h2c, pivots = _clusters(c, rng)
    prompts = [_prompt(c, seed * 64 + b) for b in range(c["batch"])]
    layers = [_layer_inputs(c, h2c, prompts, seed * 16 + x) for x in range(c.get("layers", 1))]
    q, k, _ = layers[0]
    nqb, b, heads, maps = c["seq"] // c["block"], c["batch"], c["q_heads"], len(pivots)
    shape = sp.shape_of(q, k, None, c["block"])
    s = {"case": c, "shape": shape, "layers": layers, "h2c": h2c, "pivots": pivots, "heads": list(range(heads)),
         "o": [torch.zeros_like(q) for _ in layers]}

    def new(dtype, *size):
        return torch.empty(size, dtype=dtype, device="cuda")

    need = sp.sp_workspace_bytes(shape, heads if kind == "dense" else 0 if kind == "lists" else maps)
    if kind == "slash":
        need = sp.sp_vs_token_workspace_bytes(shape, heads)
    elif kind == "lists":
        s["idx"], s["cnt"], s["maps"] = _caller_lists(c, rng)
        s["map_of"] = [h * s["maps"] // heads for h in range(heads)]
    elif kind == "dense":
        s["scores"] = new(torch.float32, b, heads, nqb, nqb)
    else:
        s["idx"], s["cnt"] = new(torch.int32, b, maps, nqb, nqb), new(torch.int32, b, maps, nqb)
        s["scores"] = new(torch.float32, b, maps, nqb, nqb) if c.get("scores") or kind == "stack" else None
    if kind in ("gated", "stack"):
        s["a_hat"], s["dist"] = new(torch.float32, b, heads, nqb), new(torch.float32, b, heads, 2)
        s["role"] = [new(torch.int32, b, heads) for _ in layers]
    if kind == "stack":
        s["valid"], s["a_tilde"] = new(torch.int32, b, maps), new(torch.float32, b, maps, nqb)
        s["dict"] = sp.pattern_dict_of(s["valid"], s["a_tilde"], s["idx"], s["cnt"])
        s["mode"], s["vs_idx"], s["vs_cnt"] = sp.SP_FALLBACK_DENSE, None, None
        if c["fallback"] == "tokens":
            s["mode"] = sp.SP_FALLBACK_VERTICAL_SLASH_TOKEN
            need += sp.sp_vs_token_workspace_bytes(shape, heads)
        elif c["fallback"] == "blocks":
            s["mode"] = sp.SP_FALLBACK_VERTICAL_SLASH
            need += sp.sp_vs_workspace_bytes(shape, heads)
            s["vs_idx"], s["vs_cnt"] = new(torch.int32, b, heads, nqb, nqb), new(torch.int32, b, heads, nqb)
    s["ws"] = new(torch.uint8, need)
    return s


def run(s):
    c, shape, ws = s["case"], s["shape"], s["ws"]
    kind, gamma = c["kind"], c["gamma"]
    q, k, v = s["layers"][0]
    o = s["o"][0]
    if kind == "layer":
        sp.sp_prefill_layer(shape, q, k, v, s["h2c"], s["pivots"], gamma, o, s["scores"], s["idx"], s["cnt"], ws)
        return {"o": o, "scores": s["scores"], "idx": s["idx"], "cnt": s["cnt"]}
    if kind == "printed":
        sp.sp_prefill_layer_modes(shape, q, k, v, s["h2c"], s["pivots"], gamma, sp.SP_SCORE_MEAN_LOGIT,
                                  sp.SP_SELECT_GLOBAL, o, None, s["idx"], s["cnt"], ws)
        return {"o": o, "idx": s["idx"], "cnt": s["cnt"]}
    if kind == "gated":
        sp.sp_prefill_layer_gated(shape, q, k, v, s["h2c"], s["pivots"], gamma, c["delta"], c["tau"],
                                  sp.SP_SCORE_BLOCK_MASS, sp.SP_SELECT_PER_ROW, o, None, s["idx"], s["cnt"], s["a_hat"],
                                  s["dist"], s["role"][0], ws)
        return {"o": o, "idx": s["idx"], "cnt": s["cnt"], "dist": s["dist"], "role": s["role"][0]}
    if kind == "stack":
        s["valid"].zero_()  # a new prompt starts with an empty dictionary
        for x, (q, k, v) in enumerate(s["layers"]):
            sp.sp_prefill_layer_dict(shape, q, k, v, s["h2c"], gamma, c["delta"], c["tau"], sp.SP_SCORE_BLOCK_MASS,
                                     sp.SP_SELECT_PER_ROW, s["dict"], s["o"][x], s["scores"], s["role"][x], s["a_hat"],
                                     s["dist"], ws, fallback_mode=s["mode"], vs_idx=s["vs_idx"], vs_cnt=s["vs_cnt"])
        return {"o": s["o"], "role": s["role"], "valid": s["valid"], "dist": s["dist"]}
    if kind == "slash":
        sp.sp_vertical_slash_attn(shape, q, k, v, s["heads"], gamma, True, o, None, None, ws)
        return o
    if kind == "dense":
        sp.sp_dense_attn_with_block_scores(shape, q, k, v, s["heads"], o, s["scores"], ws)
        return {"o": o, "scores": s["scores"]}
    sp.sp_block_sparse_attn(shape, q, k, v, s["heads"], s["map_of"], s["idx"], s["cnt"], s["maps"], o, ws)
    return o


# ------------------------------------------------------------------------------------------------ work
def _pairs(c):
    """(query, key) pairs that one pass attends to.  What the patterns keep depends on the data; the shares below are
    what these inputs keep at a long prompt (of the causal pairs), and a pattern never keeps less than the window of a
    few blocks per row that the forced blocks and the topics' segments give a short one."""
    n, heads, maps = c["seq"], c["q_heads"], c["q_heads"] // c["cluster"]
    full = n * (n + 1) / 2.0
    shared = full * min(1.0, (0.16 if c["gamma"] > 0.92 else 0.11) + 7.0 * c["block"] / n)
    diffuse = full * max(0.2, 0.34 + 0.066 * math.log2(n / 8192))   # heads that pass the sparsity test of the gate
    slash = full * min(1.0, (0.19 if c["gamma"] > 0.92 else 0.13) + 8.0 * c["block"] / n)
    if c["kind"] == "dense":
        pairs = heads * full
    elif c["kind"] == "lists":
        pairs = heads * full * min(1.0, 1.0 / 12 + 32.0 * c["block"] / n)
    elif c["kind"] == "slash":
        pairs = heads * slash
    elif c["kind"] in ("layer", "printed"):
        pairs = maps * full + (heads - maps) * shared
    else:
        layers = c.get("layers", 1)
        if c["spread"]:
            share = diffuse
        elif c["delta"] > 1:
            share = shared
        else:
            share = slash if c.get("fallback") in ("tokens", "blocks") else full
        pairs = maps * full + (layers * heads - maps) * share
    return c["batch"] * pairs


def work(case):
    """q, k, v read once and the outputs written once; two products of head_dim per attended pair."""
    c = case
    layers, nqb, maps = c.get("layers", 1), c["seq"] // c["block"], c["q_heads"] // c["cluster"]
    size = layers * c["batch"] * c["seq"] * c["head_dim"] * 2 * (2 * c["q_heads"] + 2 * c["kv_heads"])
    square = c["batch"] * nqb * nqb * 4
    if c["kind"] == "dense":
        size += c["q_heads"] * square
    elif c["kind"] != "slash":
        size += maps * square * (2 if c.get("scores") else 1)
    return {"bytes": float(size), "flops": 4.0 * c["head_dim"] * _pairs(c)}


def tolerance(case):
    # bf16 outputs from bf16 weights in the second product: against sums in 64 bits the outputs of these inputs are off by
    # 1.7e-3 (2-norm) and 8e-3 (largest, over the value or the rms), most of it the rounding of the output itself.
    if case["kind"] in ("dense", "lists"):
        return {"rel": 7e-3, "max": 0.04}
    # A pattern is a cut in sorted fp32 sums: another order of summation moves single blocks or keys in or out, each of
    # them a small share of its row but not of every query of the row.
    return {"rel": 7e-3, "max": 0.5, "differ": 5e-3}
